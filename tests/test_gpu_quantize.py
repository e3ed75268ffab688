"""GPU check of vq_quantize_columns (Algorithm 1, Sec. 3.1) against the CPU oracle.  The loop decides integers from
floating-point distances and several summation orders are legitimate, so the check is one of validity, complete in both
directions: (a) every chosen index is a nearest centroid, within EPS, of the column as the GPU itself propagated it (T),
checked in fp64; (b) T is what the algorithm's recurrence gives for the GPU's own choices, replayed by the oracle in fp64;
(c) the quantized weights are exactly what the indices restore; (d) the second-order loss is within a stated factor of
the loss of the oracle's own run."""
import numpy as np
import pytest

import oracle
import vq_synth as s

pytestmark = pytest.mark.gpu

EPS = 1e-4            # a chosen centroid may be this much (relative) farther than the nearest one: binary32 distances
TOL_T = 1e-4          # max |T_gpu - T_replayed| <= TOL_T * RMS(W): binary32 updates against the fp64 replay
LOSS_BAND = (0.9, 1.1)

CASES = {
    "v6_k4096_three_blocks": dict(M=384, N=300, v=6, k=4096, k_res=0, B=128),       # ragged last block of 44 columns
    "v6_res16_ragged_rows": dict(M=100, N=200, v=6, k=256, k_res=16, B=64),          # last vector of 4 rows
    "v8_k65536_tables_in_memory": dict(M=64, N=130, v=8, k=65536, k_res=0, B=128),   # 1 MB table: read through L2, not LDS
    "v4_res256_small_blocks": dict(M=33, N=70, v=4, k=256, k_res=256, B=32),
    "v12_k4096": dict(M=40, N=50, v=12, k=4096, k_res=0, B=128),
    "v1_scalar": dict(M=70, N=40, v=1, k=16, k_res=0, B=7),
    "v6_res4096_one_block": dict(M=60, N=100, v=6, k=4096, k_res=4096, B=128),
    # the one-launch loop: two and four positions a workgroup beside a cut-off one, every number of groups of 64 centroids a wave
    # holds, tables that end inside a group, entries of 8, 16 and 32 operand slots, an odd block of several
    "v6_two_positions_a_workgroup": dict(M=1603, N=40, v=6, k=256, k_res=0, B=32),
    "v2_four_positions_a_workgroup": dict(M=2051, N=24, v=2, k=16, k_res=0, B=9),
    "v6_k1025": dict(M=50, N=70, v=6, k=1025, k_res=1023, B=64),
    "v4_k300": dict(M=34, N=50, v=4, k=300, k_res=0, B=25),
    "v10_k4095_res60": dict(M=45, N=60, v=10, k=4095, k_res=60, B=31),
    "v16_k1000_res100": dict(M=40, N=40, v=16, k=1000, k_res=100, B=128),
    "v15_k4096_not_in_registers": dict(M=31, N=30, v=15, k=4096, k_res=0, B=128),
    "v5_k4000_res3000": dict(M=23, N=60, v=5, k=4000, k_res=3000, B=128),
}


def _tables(seed, k, v, k_res):
    C = s.to_fp16(s.normal(s.tensor_seed(600 + seed, 0), k * v, 0.02)).reshape(k, v)
    R = s.to_fp16(s.normal(s.tensor_seed(600 + seed, 1), k_res * v, 0.006)).reshape(k_res, v) if k_res else None
    return C, R


def _unpack(stream_bytes, bits, count):
    return np.stack([oracle.unpack_row(np.ascontiguousarray(row), bits, count) for row in stream_bytes])


def _vector_rows(M, v):
    for p in range(-(-M // v)):
        yield p, slice(p * v, min(M, p * v + v))


@pytest.mark.parametrize("name", list(CASES))
def test_quantize_columns_is_valid_both_ways(gpu_lib, name):
    import torch
    case = CASES[name]
    M, N, v, k, k_res, B = (case[n] for n in ("M", "N", "v", "k", "k_res", "B"))
    seed = list(CASES).index(name)
    W0 = s.make_weights(600 + seed, M, N)
    H = s.make_hessian(600 + seed, N)
    U = np.ascontiguousarray(np.linalg.cholesky(np.linalg.inv(H)).T, dtype=np.float32)             # upper factor of H^-1, as the GPU gets it
    C, R = _tables(seed, k, v, k_res)
    Wd = torch.from_numpy(W0.astype(np.float32)).cuda()
    idx_b, idx_res_b, T = gpu_lib.quantize_columns(Wd, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(),
                                                   torch.from_numpy(R).cuda() if k_res else None, block=B)
    torch.cuda.synchronize()
    S = -(-M // v)
    bits, bits_res = oracle.index_bits(k), oracle.index_bits(k_res) if k_res else 0
    idx_bytes = idx_b.cpu().numpy()
    idx = _unpack(idx_bytes, bits, N)
    idx_res = _unpack(idx_res_b.cpu().numpy(), bits_res, N) if k_res else None
    assert idx.shape == (S, N) and idx.max() < k
    # the stream's dwords are written whole (pad bits zero), the rest of the stride is left alone
    used = (N * bits + 31) // 32 * 4
    assert (idx_bytes[:, used:] == 0xEE).all()
    tail_bits = np.unpackbits(idx_bytes[:, :used], axis=1, bitorder="little")[:, N * bits:]
    assert not tail_bits.any()
    Tg = T.cpu().numpy().astype(np.float64)
    What = Wd.cpu().numpy().astype(np.float64)
    Cd = C.astype(np.float64)
    # (a) and (c)
    for p, rows in _vector_rows(M, v):
        ln = rows.stop - rows.start
        t = Tg[rows].T                                                          # [N][ln]
        d = ((t[:, None, :] - Cd[None, :, :ln]) ** 2).sum(2) if k * N * ln < 5e7 else None
        for n in range(N):
            dn = d[n] if d is not None else ((t[n][None, :] - Cd[:, :ln]) ** 2).sum(1)
            assert dn[idx[p, n]] <= dn.min() * (1 + EPS) + 1e-14, (name, p, n)
        q = Cd[idx[p], :ln]                                                     # [N][ln]
        if k_res:
            r = (t.astype(np.float32) - q.astype(np.float32)).astype(np.float64)   # the kernel's residual: one binary32 subtraction
            Rd = R.astype(np.float64)
            dr = ((r[:, None, :] - Rd[None, :, :ln]) ** 2).sum(2)
            chosen = dr[np.arange(N), idx_res[p]]
            assert (chosen <= dr.min(1) * (1 + EPS) + 1e-14).all(), (name, p)
            q = (C[idx[p], :ln].astype(np.float32) + R[idx_res[p], :ln].astype(np.float32)).astype(np.float16).astype(np.float64)
        assert np.array_equal(What[rows].T, q), (name, p)
    # (b) the recurrence, replayed in fp64 with the GPU's choices
    replay = oracle.quantize_columns(W0, U, C, R, block=B, given=(idx, idx_res))
    rms = np.sqrt((W0 ** 2).mean())
    assert np.abs(replay["T"] - Tg).max() <= TOL_T * rms, (name, np.abs(replay["T"] - Tg).max() / rms)
    assert np.array_equal(replay["What"], What)
    # (d) the loss the algorithm is after
    own = oracle.quantize_columns(W0, U, C, R, block=B)
    def loss(Wq):
        d = W0 - Wq
        return np.einsum("on,nm,om->", d, H, d)
    ratio = loss(What) / loss(own["What"])
    assert LOSS_BAND[0] <= ratio <= LOSS_BAND[1], (name, ratio)
    print("%s: indices equal to the oracle's own run: %.4f, max |T - replay| / rms %.2e, loss ratio %.4f"
          % (name, (idx == own["idx"]).mean(), np.abs(replay["T"] - Tg).max() / rms, ratio))


# Sizes and numbers at which the one-launch loop takes other paths: three and four positions a workgroup, sixteen groups of wide entries beside a
# residual table, weights so large that they do not scale into binary16 (every distance is computed), a diagonal whose
# reciprocal is not used.  Bounds: as above; with weights 2^24 times larger than the centroids all distances agree to 2^-23 or so, and
# EPS covers that.
PATHS = {
    "v6_three_positions": dict(M=3100, N=21, v=6, k=300, k_res=0, B=16),
    "v7_k1500_res900": dict(M=45, N=50, v=7, k=1500, k_res=900, B=33),
    "v12_k3000_two_positions": dict(M=3090, N=18, v=12, k=3000, k_res=0, B=16),
    "weights_out_of_scale": dict(M=40, N=40, v=6, k=256, k_res=16, B=32, w_scale=2.0 ** 24),
    "diagonal_out_of_range": dict(M=40, N=40, v=6, k=256, k_res=0, B=32, h_scale=2.0 ** -100),
}


@pytest.mark.parametrize("name", list(PATHS))
def test_quantize_columns_paths(gpu_lib, name):
    import torch
    case = PATHS[name]
    M, N, v, k, k_res, B = (case[n] for n in ("M", "N", "v", "k", "k_res", "B"))
    seed = 80 + list(PATHS).index(name)
    W0 = (s.make_weights(600 + seed, M, N).astype(np.float32) * case.get("w_scale", 1.0)).astype(np.float32)
    H = s.make_hessian(600 + seed, N) * case.get("h_scale", 1.0)
    U = np.ascontiguousarray(np.linalg.cholesky(np.linalg.inv(H)).T, dtype=np.float32)
    C, R = _tables(seed, k, v, k_res)
    Wd = torch.from_numpy(W0).cuda()
    idx_b, idx_res_b, T = gpu_lib.quantize_columns(Wd, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(),
                                                   torch.from_numpy(R).cuda() if k_res else None, block=B)
    torch.cuda.synchronize()
    idx = _unpack(idx_b.cpu().numpy(), oracle.index_bits(k), N)
    idx_res = _unpack(idx_res_b.cpu().numpy(), oracle.index_bits(k_res), N) if k_res else None
    Tg = T.cpu().numpy().astype(np.float64)
    Cd = C.astype(np.float64)
    for p, rows in _vector_rows(M, v):
        ln = rows.stop - rows.start
        t = Tg[rows].T
        d = ((t[:, None, :] - Cd[None, :, :ln]) ** 2).sum(2)
        assert (d[np.arange(N), idx[p]] <= d.min(1) * (1 + EPS) + 1e-14).all(), (name, p)
        if k_res:
            r = (t.astype(np.float32) - Cd[idx[p], :ln].astype(np.float32)).astype(np.float64)
            dr = ((r[:, None, :] - R.astype(np.float64)[None, :, :ln]) ** 2).sum(2)
            assert (dr[np.arange(N), idx_res[p]] <= dr.min(1) * (1 + EPS) + 1e-14).all(), (name, p)
    replay = oracle.quantize_columns(W0.astype(np.float64), U, C, R, block=B, given=(idx, idx_res))
    rms = np.sqrt((W0.astype(np.float64) ** 2).mean())
    assert np.abs(replay["T"] - Tg).max() <= TOL_T * rms, (name, np.abs(replay["T"] - Tg).max() / rms)
    assert np.array_equal(replay["What"], Wd.cpu().numpy().astype(np.float64))


# Where the search has to tell more from less: every entry twice, entries that differ in their last bits, a last position of one or two
# rows (in one or two dimensions many entries are about as near), vectors of one to three elements, weights beyond binary16's range.
TIGHT = {
    "every_entry_twice": dict(M=36, N=40, v=6, k=512, k_res=128, B=32, table="twice"),
    "every_entry_twice_4096": dict(M=30, N=24, v=6, k=4096, k_res=0, B=32, table="twice"),
    "last_bits": dict(M=48, N=40, v=8, k=1024, k_res=0, B=32, table="near"),
    "last_bits_4096_res": dict(M=30, N=24, v=6, k=4096, k_res=4096, B=16, table="near"),
    "one_row_left": dict(M=25, N=71, v=6, k=4096, k_res=256, B=64),
    "one_row_left_wide": dict(M=33, N=40, v=16, k=1024, k_res=0, B=40),
    "one_row_left_v12": dict(M=25, N=40, v=12, k=4096, k_res=0, B=40),
    "one_row_left_v8": dict(M=9, N=60, v=8, k=3000, k_res=200, B=64),
    "two_rows_left": dict(M=20, N=60, v=6, k=4096, k_res=4096, B=64),
    "two_rows_left_v12": dict(M=26, N=40, v=12, k=4096, k_res=0, B=40),
    "three_rows_left": dict(M=21, N=60, v=6, k=4096, k_res=0, B=64),
    "v1": dict(M=40, N=40, v=1, k=1024, k_res=60, B=32),
    "v2": dict(M=41, N=40, v=2, k=4096, k_res=0, B=32),
    "v3": dict(M=3100, N=20, v=3, k=2000, k_res=0, B=32),
    "one_row_left_out_of_scale": dict(M=25, N=40, v=6, k=4096, k_res=16, B=32, w_scale=2.0 ** 20),
}


# What a block leaves to the columns beyond the next one is applied beside the next block's columns, 128 columns a wave and eight rows of H^-1 a step:
# widths that end inside a pair of columns, inside 128 of them, in the first and in later turns of the four waves; blocks that are not whole
# steps; one to four positions a workgroup and a cut-off one; tables that leave too little LDS for a block of 128.
LATER = {
    "one_column_beyond": dict(M=13, N=257, v=6, k=64, k_res=0, B=128),
    "odd_pair": dict(M=13, N=385, v=6, k=64, k_res=16, B=128),
    "two_turns_two_positions": dict(M=1603, N=905, v=6, k=16, k_res=0, B=128),
    "three_positions": dict(M=3100, N=300, v=6, k=16, k_res=0, B=64),
    "four_positions": dict(M=4203, N=261, v=4, k=16, k_res=0, B=64),
    "v5_in_six": dict(M=1604, N=300, v=5, k=64, k_res=0, B=96),
    "v16_two_positions": dict(M=4200, N=150, v=16, k=16, k_res=0, B=40),
    "block_of_three": dict(M=20, N=150, v=6, k=64, k_res=0, B=3),
    "block_of_100": dict(M=20, N=420, v=8, k=64, k_res=0, B=100),
    "many_turns_of_a_short_block": dict(M=7, N=1500, v=6, k=16, k_res=0, B=8),
    "v12_smaller_block_than_asked": dict(M=30, N=300, v=12, k=4096, k_res=200, B=128),
}


@pytest.mark.parametrize("name", list(LATER))
def test_quantize_columns_later_columns(gpu_lib, name):
    import torch
    case = LATER[name]
    M, N, v, k, k_res, B = (case[n] for n in ("M", "N", "v", "k", "k_res", "B"))
    seed = 160 + list(LATER).index(name)
    W0 = s.make_weights(600 + seed, M, N)
    H = s.make_hessian(600 + seed, N)
    U = np.ascontiguousarray(np.linalg.cholesky(np.linalg.inv(H)).T, dtype=np.float32)
    C, R = _tables(seed, k, v, k_res)
    Wd = torch.from_numpy(W0.astype(np.float32)).cuda()
    idx_b, idx_res_b, T = gpu_lib.quantize_columns(Wd, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(),
                                                   torch.from_numpy(R).cuda() if k_res else None, block=B)
    torch.cuda.synchronize()
    idx = _unpack(idx_b.cpu().numpy(), oracle.index_bits(k), N)
    idx_res = _unpack(idx_res_b.cpu().numpy(), oracle.index_bits(k_res), N) if k_res else None
    replay = oracle.quantize_columns(W0, U, C, R, block=B, given=(idx, idx_res))
    rms = np.sqrt((W0 ** 2).mean())
    assert np.abs(replay["T"] - T.cpu().numpy().astype(np.float64)).max() <= TOL_T * rms
    assert np.array_equal(replay["What"], Wd.cpu().numpy().astype(np.float64))


# Later columns of which a whole number of 128s and one are left, which is the first of a group of 128: it once went with the last of the group before,
# another wave's (385, 513, 641 of the block's end) or a later turn's (769, 1025, 833); one left alone (257); and more of them than a block has columns for
# steps, whose rest follows at its end (4481).
ONE_MORE = {
    "left_alone": dict(M=13, N=257, v=6, k=64, k_res=0, B=128),
    "another_wave": dict(M=13, N=641, v=6, k=64, k_res=0, B=128),
    "later_turn": dict(M=13, N=769, v=6, k=64, k_res=16, B=128),
    "two_turns_v4_two_positions": dict(M=1603, N=1025, v=4, k=16, k_res=0, B=128),
    "blocks_of_64": dict(M=19, N=833, v=8, k=16, k_res=0, B=64),
    "blocks_of_8": dict(M=7, N=1553, v=6, k=16, k_res=0, B=8),
    "rest_at_the_end": dict(M=7, N=4481, v=6, k=16, k_res=0, B=128),
}

# Blocks of up to eight columns: all four keeping waves have a step of the later update in every block.
SHORTEST = {
    "one_column": dict(M=25, N=1100, v=6, k=16, k_res=0, B=1),
    "seven": dict(M=25, N=1101, v=6, k=64, k_res=16, B=7),
    "eight_two_positions": dict(M=1603, N=700, v=4, k=16, k_res=0, B=8),
}


@pytest.mark.parametrize("name", list(ONE_MORE) + list(SHORTEST))
def test_quantize_columns_one_more_than_whole_groups(gpu_lib, name):
    import torch
    case = {**ONE_MORE, **SHORTEST}[name]
    M, N, v, k, k_res, B = (case[n] for n in ("M", "N", "v", "k", "k_res", "B"))
    seed = 190 + (list(ONE_MORE) + list(SHORTEST)).index(name)
    W0 = s.make_weights(600 + seed, M, N)
    U = np.triu(np.random.default_rng(seed).standard_normal((N, N), dtype=np.float32) * np.float32(0.02), 1) + np.eye(N, dtype=np.float32)
    C, R = _tables(seed, k, v, k_res)
    Wd = torch.from_numpy(W0.astype(np.float32)).cuda()
    idx_b, idx_res_b, T = gpu_lib.quantize_columns(Wd, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(),
                                                   torch.from_numpy(R).cuda() if k_res else None, block=B)
    torch.cuda.synchronize()
    idx = _unpack(idx_b.cpu().numpy(), oracle.index_bits(k), N)
    idx_res = _unpack(idx_res_b.cpu().numpy(), oracle.index_bits(k_res), N) if k_res else None
    replay = oracle.quantize_columns(W0, U, C, R, block=B, given=(idx, idx_res))
    rms = np.sqrt((W0 ** 2).mean())
    assert np.abs(replay["T"] - T.cpu().numpy().astype(np.float64)).max() <= TOL_T * rms
    assert np.array_equal(replay["What"], Wd.cpu().numpy().astype(np.float64))


def _tight_tables(seed, case):
    C, R = _tables(seed, case["k"], case["v"], case["k_res"])
    for T in (C, R):
        if T is None or "table" not in case:
            continue
        half = len(T) // 2
        T[half:] = T[:half] if case["table"] == "twice" else np.nextafter(T[:half], np.float16(np.inf))
    return C, R


@pytest.mark.parametrize("name", list(CASES) + list(PATHS) + list(TIGHT))
def test_quantize_columns_takes_the_first_of_the_nearest(gpu_lib, name):
    """The distance of include/vq.h is binary32 arithmetic fixed to the last bit, and T is returned in binary32: every index is the first
    one of the smallest distance from T's vector, and every residual index that of T less the main centroid (one subtraction)."""
    import torch
    case = {**CASES, **PATHS, **TIGHT}[name]
    M, N, v, k, k_res, B = (case[n] for n in ("M", "N", "v", "k", "k_res", "B"))
    seed = 120 + (list(CASES) + list(PATHS) + list(TIGHT)).index(name)
    W0 = (s.make_weights(600 + seed, M, N).astype(np.float32) * case.get("w_scale", 1.0)).astype(np.float32)
    H = s.make_hessian(600 + seed, N) * case.get("h_scale", 1.0)
    U = np.ascontiguousarray(np.linalg.cholesky(np.linalg.inv(H)).T, dtype=np.float32)
    C, R = _tight_tables(seed, case)
    Wd = torch.from_numpy(W0).cuda()
    idx_b, idx_res_b, T = gpu_lib.quantize_columns(Wd, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(),
                                                   torch.from_numpy(R).cuda() if k_res else None, block=B)
    torch.cuda.synchronize()
    idx = _unpack(idx_b.cpu().numpy(), oracle.index_bits(k), N)
    T = T.cpu().numpy()
    want = oracle.nearest_down(T, C)
    assert np.array_equal(idx, want), (name, int((idx != want).sum()), np.argwhere(idx != want)[:4].tolist())
    if k_res:
        q = C[idx].transpose(0, 2, 1).reshape(-1, N)[:M].astype(np.float32)             # [positions][N][v] -> rows
        want = oracle.nearest_down(T - q, R)
        idx_res = _unpack(idx_res_b.cpu().numpy(), oracle.index_bits(k_res), N)
        assert np.array_equal(idx_res, want), (name, int((idx_res != want).sum()), np.argwhere(idx_res != want)[:4].tolist())


def test_quantize_columns_divides(gpu_lib):
    """E is a division, rounded once, down to the subnormal numbers and for diagonals far from one.  The factor couples columns 2 i and
    2 i + 1 alone, with 1, and the odd columns are zeros: T there is 0 - E of the column before."""
    import torch
    M, N = 72, 512
    rng = np.random.default_rng(5)
    W = np.zeros((M, N), dtype=np.float32)
    exponent = rng.integers(-148, -60, (M, N // 2))
    exponent[:, ::4] = rng.integers(-30, -4, (M, N // 8))
    W[:, ::2] = (rng.uniform(1, 2, (M, N // 2)) * 2.0 ** exponent * rng.choice([-1.0, 1.0], (M, N // 2))).astype(np.float32)
    W[::7, ::2] = -0.0
    U = np.zeros((N, N), dtype=np.float32)
    diagonal = rng.uniform(1, 2, N).astype(np.float32)
    diagonal[64:128] *= np.float32(2.0) ** rng.integers(-39, 39, 64).astype(np.float32)
    diagonal[128:160] *= -1.0
    U[np.arange(N), np.arange(N)] = diagonal
    U[np.arange(0, N, 2), np.arange(1, N, 2)] = 1.0
    C = np.zeros((16, 6), dtype=np.float16)
    C[1:] = s.to_fp16(s.normal(77, 15 * 6, 0.02)).reshape(15, 6)
    Wd = torch.from_numpy(W).cuda()
    idx_b, _, T = gpu_lib.quantize_columns(Wd, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(), None, block=128)
    torch.cuda.synchronize()
    idx = _unpack(idx_b.cpu().numpy(), 4, N)
    q = C[idx].transpose(0, 2, 1).reshape(-1, N)[:M].astype(np.float32)
    T = T.cpu().numpy()
    assert np.array_equal(T[:, ::2], W[:, ::2])
    with np.errstate(under="ignore", over="ignore"):
        E = (W - q)[:, ::2] / diagonal[::2]                          # (numpy divides binary32 numbers with one rounding)
    got = T[:, 1::2]
    wrong = got != -E
    assert not wrong.any(), (int(wrong.sum()), W[:, ::2][wrong][:4], got[wrong][:4], -E[wrong][:4])
    assert (E != 0).mean() > 0.5 and (np.abs(E[E != 0]) < 2.0 ** -126).any()


def test_quantize_columns_restores_through_the_layer_path(gpu_lib):
    """The streams it writes are a layer of orientation 1: vq_dequant restores exactly the quantized weights it returned."""
    import torch
    M, N, v, k, k_res = 90, 136, 6, 4096, 256
    W0 = s.make_weights(650, M, N)
    U = np.ascontiguousarray(np.linalg.cholesky(np.linalg.inv(s.make_hessian(650, N))).T, dtype=np.float32)
    C, R = _tables(50, k, v, k_res)
    Wd = torch.from_numpy(W0.astype(np.float32)).cuda()
    idx_b, idx_res_b, _ = gpu_lib.quantize_columns(Wd, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(), torch.from_numpy(R).cuda(), block=128, want_T=False)
    again = torch.from_numpy(W0.astype(np.float32)).cuda()
    idx_b2, idx_res_b2, _ = gpu_lib.quantize_columns(again, torch.from_numpy(U).cuda(), torch.from_numpy(C).cuda(), torch.from_numpy(R).cuda(), block=128, want_T=False)
    torch.cuda.synchronize()
    assert torch.equal(idx_b, idx_b2) and torch.equal(idx_res_b, idx_res_b2) and torch.equal(Wd, again)      # deterministic
    L = s.VQLayer("quantized", M, N, v, k, k_res, orientation=1)
    L.codebook, L.codebook_res = C, R
    L.idx, L.idx_res = idx_b.cpu().numpy(), idx_res_b.cpu().numpy()
    restored = gpu_lib.dequant(gpu_lib.DeviceLayer(L))
    torch.cuda.synchronize()
    assert np.array_equal(restored.float().cpu().numpy(), Wd.cpu().numpy())
    assert np.array_equal(oracle.dequant(L).astype(np.float32), Wd.cpu().numpy())


def test_quantize_columns_rejects_bad_arguments(gpu_lib):
    import torch
    W = torch.zeros((12, 16), dtype=torch.float32, device="cuda")
    Hi = torch.eye(16, dtype=torch.float32, device="cuda")
    C = torch.zeros((16, 6), dtype=torch.float16, device="cuda")
    idx = torch.zeros((2, 16), dtype=torch.uint8, device="cuda")
    need = gpu_lib.vq_quantize_columns_workspace_bytes(12, 6, 16, 0)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    def call(**kw):
        a = dict(W=W.data_ptr(), ldw=16, rows=12, cols=16, Hinv=Hi.data_ptr(), ldh=16, cb=C.data_ptr(), v=6, k=16, cbr=None, k_res=0, block=8,
                 idx=idx.data_ptr(), stride=16, idxr=None, strider=0, T=None, ldt=0, ws=ws.data_ptr(), wsb=need)
        a.update(kw)
        return gpu_lib.vq_quantize_columns(a["W"], a["ldw"], a["rows"], a["cols"], a["Hinv"], a["ldh"], a["cb"], a["v"], a["k"], a["cbr"], a["k_res"],
                                           a["block"], a["idx"], a["stride"], a["idxr"], a["strider"], a["T"], a["ldt"], a["ws"], a["wsb"], None)
    assert call() == gpu_lib.VQ_OK
    assert call(W=None) == gpu_lib.VQ_ERR_NULL and call(idx=None) == gpu_lib.VQ_ERR_NULL
    assert call(block=0) == gpu_lib.VQ_ERR_SHAPE and call(block=129) == gpu_lib.VQ_ERR_SHAPE and call(ldw=15) == gpu_lib.VQ_ERR_SHAPE
    assert call(k_res=16) == gpu_lib.VQ_ERR_NULL
    assert call(stride=4) == gpu_lib.VQ_ERR_SHAPE and call(stride=24) == gpu_lib.VQ_ERR_ALIGNMENT
    assert call(wsb=need - 1) == gpu_lib.VQ_ERR_WORKSPACE and call(ws=None) == gpu_lib.VQ_ERR_WORKSPACE
    torch.cuda.synchronize()
