"""The index arithmetic that kernels share with this host build (csrc/q8_index.h): every piece of work is dealt out
exactly once, and every address that follows from it lies inside the array it reads."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    out = os.path.join(ROOT, "tests", "support", "_build")
    os.makedirs(out, exist_ok=True)
    so = os.path.join(out, "q8_index_host.so")
    subprocess.run(["gcc", "-O2", "-std=c11", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_1804_05038_amd", "csrc"),
                    os.path.join(ROOT, "tests", "support", "q8_index_host.c"), "-o", so], check=True)
    return ctypes.CDLL(so)


def _ints(n):
    return (ctypes.c_int * n)()


@pytest.mark.parametrize("first", [0, 1, 90, 100000])
@pytest.mark.parametrize("lens", [[30, 30, 30], [1], [7, 0, 0, 5, 0], [0, 0], [60] * 200, [1] * 3, [1024] * 1000])
@pytest.mark.parametrize("blocks", [1, 2, 97, 384, 768])
def test_position_runs_cover_the_sentences_of_a_group_once(lib, first, lens, blocks):
    """Offsets that begin at any value: the runs are back to back from the first position to the last, none longer
    than the others by more than one, and each begins inside one of the sentences."""
    off = np.concatenate([[first], first + np.cumsum(lens)]).astype(np.int32)
    pos, end = _ints(blocks), _ints(blocks)
    lib.q8x_position_runs(off.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), len(lens), blocks, pos, end)
    pos, end = np.array(pos[:]), np.array(end[:])
    assert pos[0] == off[0] and end[-1] == off[-1] and (pos[1:] == end[:-1]).all()
    assert (end >= pos).all() and np.ptp(end - pos) <= 1
    for p in pos[pos < end]:
        assert ((off[:-1] <= p) & (p < off[1:])).sum() == 1


@pytest.mark.parametrize("row_groups,slot_tiles,blocks", [(1, 1, 1), (1, 8, 1), (782, 1, 256), (782, 8, 64), (995, 7, 51), (3, 5, 3), (1024, 8, 8)])
def test_panel_runs_cover_the_units_once(lib, row_groups, slot_tiles, blocks):
    waves = 8
    u0, u1, rp0 = (_ints(blocks * waves) for _ in range(3))
    lib.q8x_panel_runs(row_groups, slot_tiles, blocks, waves, u0, u1, rp0)
    u0, u1, rp0 = (np.array(v[:]) for v in (u0, u1, rp0))
    assert u0[0] == 0 and u1[-1] == row_groups * slot_tiles and (u0[1:] == u1[:-1]).all() and np.ptp(u1 - u0) <= 1
    assert (rp0.reshape(blocks, waves) == (u0.reshape(blocks, waves)[:, :1] // slot_tiles)).all()


@pytest.mark.parametrize("first,units", [(0, 0), (7, 1), (3, 7), (100, 8), (5, 15), (0, 16), (11, 97), (40000, 131072)])
def test_panel_wave_runs_cover_a_blocks_units_once(lib, first, units):
    """Back to back from the block's first unit to its last, the first four waves' share of all 9 / 16 to within a unit."""
    u0, u1 = _ints(8), _ints(8)
    lib.q8x_panel_wave_runs(first, first + units, u0, u1)
    u0, u1 = np.array(u0[:]), np.array(u1[:])
    assert u0[0] == first and u1[-1] == first + units and (u0[1:] == u1[:-1]).all() and (u1 >= u0).all()
    assert abs((u1[:4] - u0[:4]).sum() - units * 9 / 16) <= 1 and (u1 - u0).max() <= units * 9 / 64 + 1


@pytest.mark.parametrize("ks", [16, 20])
@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 48, 49, 64, 65, 1009, 50000, 50016, 50032, 50048])
def test_panel_weights_lie_inside_the_packed_matrix(lib, ks, rows):
    """Every byte that a wave asks for, for each half that it can come to (one group past the last: a wave without units),
    is inside the rows / 16 tiles of 32 ks bytes times 16 that are there, and where the tile exists it is the right one:
    row r's piece (k step s, half h) lies at tile r / 16, 64-byte block s / 2, piece 2 (s % 2) + h."""
    ntiles = (rows + 15) // 16
    groups = (rows + 63) // 64
    at = (ctypes.c_uint * (64 * ks))()
    lane, step = np.arange(64)[:, None], np.arange(ks)[None, :]
    for half in {0, 1, *range(max(0, 2 * groups - 3), 2 * groups + 2)}:
        lib.q8x_panel_weights(half, ks, ntiles, at)
        got = np.array(at[:], dtype=np.int64).reshape(64, ks)
        assert got.min() >= 0 and got.max() + 16 <= ntiles * 16 * 32 * ks
        row = 32 * half + (lane & 31)
        want = ((row >> 4) * (ks // 2) + (step >> 1)) * 1024 + (2 * (step & 1) + (lane >> 5)) * 256 + (row & 15) * 16
        assert (got == want)[np.broadcast_to(row < 16 * ntiles, got.shape)].all()


@pytest.mark.parametrize("ld", [512, 640])
def test_panel_plans_fit_the_lds(lib, ld):
    """Every vocabulary of up to 65536 rows times every panel of 9 to 1024 slots has a plan whose LDS is there, whose
    groups cover the slots, and whose blocks hold the biases of all rows that their runs touch."""
    lds, bias = ctypes.c_ulonglong(), ctypes.c_int()
    for n in [*range(9, 70), *range(95, 1024, 31), 256, 257, 288, 289, 320, 512, 1000, 1023, 1024]:
        lib.q8x_panel_plans(65536, 97 if n % 8 else 63, ld, n, ctypes.byref(lds), ctypes.byref(bias))
        assert 0 < lds.value <= 160 * 1024 and bias.value <= 0, (n, lds.value, bias.value)


@pytest.mark.parametrize("H", [4, 32, 36, 100, 256, 512, 516, 1000, 1024])
def test_batched_encoder_plans_fit_the_lds_of_a_plain_launch(lib, H):
    """All numbers of sentences that the entry point takes (1024): no block needs more than 64 KB with the kernel's own
    variables (144 bytes), every sentence has a slot, and there is at most a block per compute unit."""
    assert 0 < lib.q8x_enc_lds(H, 1024) <= 64 * 1024 - 256


def test_batches_that_one_launch_of_the_encoder_pays_for(lib):
    one = lib.q8x_enc_one_launch
    for H in (4, 64, 256, 512, 516, 1000, 1024):
        assert not one(H, 1, 1) and not one(H, 64, 2) and one(H, 1, 3) and one(H, 64, 3) and one(H, 200, 60)
    assert one(1024, 512, 3) and not one(1024, 513, 60) and not one(1024, 1024, 1024) and not one(516, 1024, 1024)
    assert one(512, 384, 3) and not one(512, 385, 6) and one(512, 385, 7) and one(512, 1024, 7) and not one(256, 1024, 6) and one(256, 1024, 7)


def _enc_accesses(scale_at, it):
    """What the sixteen waves of the batched encoder's block do in LDS in iteration `it` (a group of slots at a time step), as
    (interval between barriers, wave, array, index, is a write): codes in front of the first of its two barriers, products
    between them, gates behind the second, where the waves without any are in front of the next iteration's first."""
    for w in range(16):
        yield 2 * it, w, "scale", scale_at(it, w), True
        yield 2 * it, w, "codes", w, True
    for w in range(12):
        for slot in range(16):
            yield 2 * it + 1, w, "codes", slot, False
        yield 2 * it + 1, w, "sums", w, True
    for w in range(8):
        for slot in (2 * w, 2 * w + 1):
            yield 2 * it + 2, w, "scale", scale_at(it, slot), False
        for tile in range(12):
            yield 2 * it + 2, w, "sums", tile, False


def test_no_two_waves_of_the_batched_encoder_meet_in_lds(lib):
    """With several groups of slots nothing but the barriers orders the waves: between two of them, what one wave writes no
    other touches, over any run of iterations (an array of one set of scales fails this)."""
    seen, written = {}, {}
    for it in range(9):
        assert all(0 <= lib.q8x_enc_scale(it, s) < 32 for s in range(16))
        for interval, wave, array, at, write in _enc_accesses(lib.q8x_enc_scale, it):
            key = interval, array, at
            assert not (write and seen.get(key, {wave}) - {wave}), (key, wave)
            assert not (written.get(key, {wave}) - {wave}), (key, wave)
            seen.setdefault(key, set()).add(wave)
            if write:
                written.setdefault(key, set()).add(wave)


def _enc_x_accesses(lib, last):
    """The same for one group per set, where the block multiplies rows of X as well: (interval, wave, array, index, write) of a
    whole run of steps.  Rows go to LDS at the start of a step (the first one's in front), their products are made behind its second barrier."""
    for w in range(16):
        yield -2, w, "rows", (0, w ^ 8), True
        yield -2, w, "row scale", lib.q8x_enc_x_scale(0, w ^ 8), True
    for t in range(-1, last):
        at = 2 * t + 2                                       # behind step t's second barrier, in front of the next step's first
        for w in range(12):
            for slot in range(16):
                yield at, w, "rows", ((t + 1) & 1, slot), False
            yield at, w, "row sums", ((t + 1) & 1, w), True
        for w in range(16):
            yield at, w, "rows", ((t + 2) & 1, w ^ 8), True
            yield at, w, "row scale", lib.q8x_enc_x_scale(t + 2, w ^ 8), True
            yield at, w, "scale", lib.q8x_enc_scale(t + 1, w ^ 8), True
            yield at, w, "codes", w ^ 8, True
        for w in range(8) if t >= 0 else ():
            for slot in (2 * w, 2 * w + 1):
                yield at, w, "scale", lib.q8x_enc_scale(t, slot), False
                yield at, w, "row scale", lib.q8x_enc_x_scale(t, slot), False
            for tile in range(12):
                yield at, w, "sums", tile, False
                yield at, w, "row sums", (t & 1, tile), False
        for w in range(12):
            for slot in range(16):
                yield at + 1, w, "codes", slot, False
            yield at + 1, w, "sums", w, True


def test_no_two_waves_of_the_batched_encoder_meet_in_the_lds_of_x(lib):
    seen, written = {}, {}
    for interval, wave, array, at, write in sorted(_enc_x_accesses(lib, 9), key=lambda a: a[0]):
        key = interval, array, at
        assert not (write and seen.get(key, {wave}) - {wave}), (key, wave)
        assert not (written.get(key, {wave}) - {wave}), (key, wave)
        seen.setdefault(key, set()).add(wave)
        if write:
            written.setdefault(key, set()).add(wave)
    assert all(0 <= lib.q8x_enc_x_scale(it, s) < 64 for it in range(9) for s in range(16))


@pytest.mark.parametrize("xs", [4, 5])
@pytest.mark.parametrize("H", [4, 32, 256, 512, 1000, 1024])
def test_batched_encoder_with_rows_of_x_fits_the_lds(lib, H, xs):
    """160 KB of a compute unit, with 2 KB for the kernel's own variables."""
    assert 0 < lib.q8x_enc_x_lds(H, xs) <= 160 * 1024 - 2048


def test_panel_products_that_quantize_their_vectors(lib):
    """The device tests' shapes take the kernel, in the form they are listed for, and no shape takes more blocks than the rule says."""
    from test_gpu_products import QUANT_PANELS
    seen = set()
    for rows, cols, n, tiled, tiles in QUANT_PANELS:
        ld = (cols + 15) // 16 * 16
        assert lib.q8x_quant_rows(rows, ld, n) == tiles, (rows, cols, n)
        seen.add((tiles, 1 + (ld > 512) + (ld > 1024)))
    assert seen == {(t, k) for t in (1, 2, 4) for k in (1, 2, 3)}
    for n in (1, 8):
        assert lib.q8x_quant_rows(1024, 512, n) == 0 and lib.q8x_part_rows(1024, 1024, n, 1) == 0
    from test_gpu_products import PART_PANELS
    for rows, cols, n, tiled, tiles in PART_PANELS:
        assert lib.q8x_part_rows(rows, (cols + 15) // 16 * 16, n, 1) == tiles, (rows, cols, n)
    assert lib.q8x_part_rows(1024, 1024, 80, 3) == 4 and lib.q8x_part_rows(1024, 1024, 81, 3) == 0 and lib.q8x_part_rows(1024, 512, 9, 1) == 0
    assert lib.q8x_quant_rows(1024, 2064, 9) == 0 and lib.q8x_quant_rows(1024, 2048, 257) == 0 and lib.q8x_quant_rows(1024, 2048, 256) == 4


@pytest.mark.parametrize("ldx,ldh", [(16, 16), (64, 1024), (512, 1024), (624, 1008), (1024, 1024), (1040, 1024), (2000, 1008), (2048, 1024), (1024, 2048), (4096, 16)])
def test_gru_parts_cover_both_products_once(lib, ldx, ldh):
    """Every 64-byte step of either product's rows belongs to one part, and no part has more than the stages' steps."""
    columns, nx, stages, k0, steps = ctypes.c_int(), ctypes.c_int(), ctypes.c_int(), _ints(3), _ints(3)
    lib.q8x_gru_tile(1024, ldx, ldh, 64, 0, 0, ctypes.byref(columns), ctypes.byref(nx), k0, steps, ctypes.byref(stages))
    assert nx.value in (1, 2) and 2 * (stages.value - 1) < max(steps[:]) <= 2 * stages.value
    for parts, ld in ((range(nx.value), ldx), (range(nx.value, 3), ldh)):
        assert [s for p in parts for s in range(k0[p], k0[p] + steps[p])] == list(range((ld + 63) // 64))


def test_gru_tile_blocks_cover_the_vectors_in_one_round(lib):
    columns, nx, stages, k0, steps = ctypes.c_int(), ctypes.c_int(), ctypes.c_int(), _ints(3), _ints(3)
    taken = 0
    for H in (4, 32, 36, 256, 512, 1000, 1024, 2048, 8192):
        for n in (9, 32, 33, 128, 129, 350, 352, 353, 700, 1000, 1024):
            for codes in (0, 1):
                if lib.q8x_gru_tile(H, 512, 512, n, codes, 1, ctypes.byref(columns), ctypes.byref(nx), k0, steps, ctypes.byref(stages)):
                    taken += 1
                    assert 1 <= columns.value <= 4 and (H + 31) // 32 * -(-n // (32 * columns.value)) <= 256
    assert taken


def test_panel_grus_in_tiles(lib):
    """The device tests' shapes take the kernel, in the form they are listed for: one to four tiles, with codes and without."""
    from test_gpu_batch import TILE_GRUS, TILE_STEPS
    columns, nx, stages, k0, steps = ctypes.c_int(), ctypes.c_int(), ctypes.c_int(), _ints(3), _ints(3)
    pitch = lambda cols: (cols + 15) // 16 * 16
    takes = lambda I, H, n, codes, packed: lib.q8x_gru_tile(H, pitch(I), pitch(H), n, codes, packed, ctypes.byref(columns), ctypes.byref(nx), k0, steps, ctypes.byref(stages))
    for I, H, n, tiled, want in TILE_GRUS:
        assert (I, H, want) == (512, 1024, 0) or (takes(I, H, n, 0, tiled) and columns.value == want), (I, H, n)
    for E, H, A, S, beam, tiled, want in TILE_STEPS:
        assert S * beam > 336 or (E, H) != (512, 1024)       # (the kernel whose blocks exchange maxima takes up to 336)
        for I in (E, 2 * H):
            assert takes(I, H, S * beam, 1, tiled) and columns.value == want, (I, H, S, beam)
    for I, H, packed, most in ((1024, 1024, 0, 192), (1024, 1024, 1, 144), (768, 768, 1, 128), (1000, 1000, 0, 160), (2048, 2048, 0, 192), (1400, 1400, 0, 128), (620, 1000, 0, 128), (400, 400, 0, 0)):
        assert not most or not takes(I, H, most, 0, packed), (I, H)
        assert takes(I, H, most + 9, 0, packed), (I, H)
    assert {c[-1] for c in TILE_GRUS} == {0, 1, 2, 3, 4} and {c[-1] for c in TILE_STEPS} >= {2, 4}


def test_encoder_of_one_sentence_is_one_launch_from_a_number_of_words_on(lib):
    """Row-major matrices of few units need more words the longer the rows of X are; beyond 8 words every shape is one launch."""
    one = lib.q8x_enc_one_better
    for H, ldx, packed, words in ((1024, 512, 1, 5), (1024, 512, 0, 6), (1024, 448, 0, 5), (1024, 640, 1, 5), (1024, 624, 0, 6), (1024, 640, 0, 8), (1000, 624, 0, 5), (1024, 1024, 1, 8),
                                  (512, 1024, 1, 1), (256, 512, 0, 1), (256, 768, 0, 7), (64, 1024, 0, 8), (36, 1024, 0, 1)):
        assert [bool(one(H, ldx, packed, l)) for l in range(1, 12)] == [l >= words for l in range(1, 12)], (H, ldx, packed)
    assert [l for l in range(1, 8) if one(256, 640, 0, l)] == [1, 5, 6, 7]


ROUTES = ["staged", "resident", "resident 1024", "tiles of 64", "tiles of 128", "once 64 x 64", "once 128 x 32", "once 128 x 64", "once 128 x 64 trade", "stream"]


def test_panel_products_take_the_kernels_that_their_tests_name(lib):
    """The rule that q8i_gemm_jobs follows, on the shapes of the device tests: each takes the kernel it is listed for, and every
    kernel has shapes."""
    from test_gpu_products import LARGE_PANELS, WHOLE_PANELS
    seen = set()
    for rows, cols, n, tiled, route in LARGE_PANELS + WHOLE_PANELS:
        assert ROUTES[lib.q8x_panel_route(rows, (cols + 15) // 16 * 16, n, int(tiled), rows)] == route, (rows, cols, n, tiled)
        seen.add((route, tiled))
    assert {r for r, _ in seen} == set(ROUTES)
    assert {r for r, t in seen if t} == set(ROUTES) - {"staged", "resident 1024", "once 128 x 64 trade"}
    assert {r for r, t in seen if not t} == set(ROUTES) - {"tiles of 64"}
    # row by row in rows of whole 128 bytes: the K-resident blocks while they are one round, for any number of vectors
    for ld in (640, 768, 896, 1024):
        for rows, n in ((64, 9), (3072, 9), (3072, 64), (3072, 320), (8192, 33), (8192, 128)):
            assert ROUTES[lib.q8x_panel_route(rows, ld, n, 0, rows)] == "resident 1024"
            assert ROUTES[lib.q8x_panel_route(rows, ld, n, 1, rows)] == ROUTES[lib.q8x_panel_route(rows, ld - 16, n, 0, rows)] == "once 128 x 32"
        assert ROUTES[lib.q8x_panel_route(20000, ld, 9, 0, 20000)] == "once 128 x 32"
    for n in (1, 8):                                                   # the batched step of few slots has such products
        assert ROUTES[lib.q8x_panel_route(3072, 1024, n, 1, 3072)] == ROUTES[lib.q8x_panel_route(3072, 1008, n, 0, 3072)] == "once 128 x 32"
        assert ROUTES[lib.q8x_panel_route(3072, 1024, n, 0, 3072)] == "resident 1024"
        assert ROUTES[lib.q8x_panel_route(3072, 512, n, 1, 3072)] == ROUTES[lib.q8x_panel_route(3072, 2048, n, 1, 3072)] == "staged"
