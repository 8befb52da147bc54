"""Host-only checks of the HIP library: it loads, exports every symbol the headers
declare, and its pure-integer staleness functions follow Eq. 8-9 (brute force)."""
import ctypes
import os
import random
import re
import subprocess
import sys
import time

import pytest

import paper_1909_06695_amd as P
from paper_1909_06695_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    names = set()
    for h in ("ouro.h", "ouro_ops.h"):
        text = open(os.path.join(ROOT, "include", h)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(ouro_[a-z0-9_]+)\s*\(", text))
    return names


def test_library_exports_every_declared_symbol():
    L = P.lib()
    decl = declared_symbols()
    assert len(decl) >= 30
    for name in decl:
        assert hasattr(L, name), name
    assert decl == set(P.exported_symbols())        # the binding covers the whole boundary


def test_ring_depths():
    for K in range(1, 9):
        assert P.ring_depth(K, 0) == K
        assert P.ring_depth(K, K + 1) == 1
        for k in range(1, K + 1):
            assert P.ring_depth(K, k) == K - k + 1
    with pytest.raises(P.OuroError):
        P.ring_depth(3, 5)


@pytest.mark.parametrize("K", [1, 2, 3, 4, 8])
def test_slot_index_against_brute_force(K):
    """Simulate the rings literally: a slot read at iteration t must still hold the
    gradient of iteration t-K+k (Eq. 8) / t-K+1 (Eq. 9), i.e. no later write has landed on
    it, and a zero gradient is prescribed exactly while that index is negative."""
    stores = {i: [None] * P.ring_depth(K, i) for i in range(K + 2)}
    for t in range(3 * K + 5):
        for i in range(K + 2):                       # backward of iteration t writes
            slot, tau = P.slot_index(K, i, t, True)
            assert tau == t and 0 <= slot < len(stores[i])
            stores[i][slot] = t
        for i in range(K + 2):                       # updates of iteration t read
            slot, tau = P.slot_index(K, i, t, False)
            want = t if i == K + 1 else (t - K + 1 if i == 0 else t - K + i)
            if want < 0:
                assert (slot, tau) == (-1, -1)
            else:
                assert tau == want and stores[i][slot] == want, (K, i, t)


def test_config_validation_is_host_side():
    good = dict(n_layer=2, d_model=64, n_head=2, d_head=32, d_ff=256, vocab=256, seq_len=32, batch=4, n_module=2)
    assert P.query_arena_bytes(P.make_config(**good)) > 0
    bad = [dict(n_head=3), dict(d_model=63, n_head=1, d_head=63), dict(n_module=3), dict(n_module=0),
           dict(mem_len=4), dict(dtype=2), dict(optimizer=5), dict(layers_per_module=[2, 1]),
           dict(layers_per_module=[2, 0]), dict(vocab=1), dict(rel_pos=2), dict(schedule=2), dict(schedule=-1),
           dict(dropout=1.0), dict(dropout=-0.1), dict(dropout=float("nan"))]
    for b in bad:
        kw = dict(good); kw.update(b)
        with pytest.raises(P.OuroError) as e:
            P.query_arena_bytes(P.make_config(**kw))
        assert e.value.code == binding.E_CONFIG, b
    # bf16 + Adam needs more arena than fp32 + SGD of the same shape? (shadow + moments vs half-size activations)
    a = P.query_arena_bytes(P.make_config(**good))
    b = P.query_arena_bytes(P.make_config(**dict(good, optimizer=1)))
    assert b > a
    # the stored-input schedule keeps module inputs instead of rings of gradients: for a deep
    # pipeline of wide layers that is the smaller arena (the point of the memory paragraph)
    big = dict(n_layer=8, d_model=256, n_head=4, d_head=64, d_ff=1024, vocab=512, seq_len=64, batch=2, n_module=8, dtype=1, optimizer=1)
    assert P.query_arena_bytes(P.make_config(**dict(big, schedule=1))) < P.query_arena_bytes(P.make_config(**big))


def test_create_model_rejects_bad_arena_without_touching_it():
    cfg = P.make_config(n_layer=1, d_model=8, n_head=2, d_head=4, d_ff=8, vocab=8, seq_len=4, batch=1)
    h = ctypes.c_void_p()
    rc = P.lib().ouro_create_model(ctypes.byref(cfg), None, 0, None, ctypes.byref(h))
    assert rc == binding.E_ARENA and not h.value
    rc = P.lib().ouro_create_model(ctypes.byref(cfg), ctypes.c_void_p(256), 16, None, ctypes.byref(h))
    assert rc == binding.E_ARENA and not h.value


@pytest.mark.parametrize("dtype,esz", [(0, 4), (1, 2)])
def test_contraction_operands_end_at_their_last_element(dtype, esz):
    """What the buffer descriptors of the contraction kernels let through ends with the operand's last element, also where
    the operand is the last column block of a wider matrix: rows * ld from the block's base would run past that matrix."""
    f = P.lib().ouro_op_gemm_operand_bytes
    for rows, ld in [(1, 1600), (33, 1600), (2331, 2304), (7, 41)]:
        for cols in {1, 8, ld // 2, ld}:
            off = ld - cols
            assert f(dtype, rows, cols, ld) + off * esz == rows * ld * esz
    assert f(dtype, 0, 8, 8) == 0
    # sizes beyond 32 bits do not wrap
    assert f(dtype, 1 << 20, 8, 1 << 14) == esz * (((1 << 20) - 1) * (1 << 14) + 8)


def plan(dtype, tA, tB, M, N, K, acc=0):
    tile, splits = ctypes.c_int(), ctypes.c_int()
    assert P.lib().ouro_op_gemm_plan(dtype, tA, tB, M, N, K, acc, ctypes.byref(tile), ctypes.byref(splits)) == 0
    return tile.value, splits.value


@pytest.mark.parametrize("M,N,K,big", [(256, 4232, 7488, False), (616, 1720, 4544, False), (4472, 5312, 3200, False), (8192, 1024, 50304, True)])
def test_split_contractions_price_their_atomic_adds(M, N, K, big):
    """256x256 tiles (14) pay for an accumulating product only where the contraction is long against the output's adds; the
    others took 1.2 to 1.8 times as long on them as on 128-wide tiles (11, 12)."""
    for tA, tB in ((1, 0), (0, 1)):
        tile, splits = plan(1, tA, tB, M, N, K, 1)
        assert tile in ((14,) if big else (11, 12)) and 1 <= splits <= max(1, K // 256)


@pytest.mark.parametrize("tA,tB", [(0, 0), (0, 1), (1, 0)])
def test_tiles_of_few_tile_products(tA, tB):
    """Up to one round of 64x64 tiles (15), but the register-prefetch kernel (13) for long contractions of a column-form
    operand with both sides long, which the 64x64 tiles made slower."""
    assert plan(1, tA, tB, 768, 1024, 1024)[0] == 15 and plan(1, tA, tB, 448, 4096, 8192)[0] == 15
    assert plan(1, tA, tB, 1344, 528, 7552)[0] == 15
    assert plan(1, tA, tB, 1088, 1496, 8192)[0] == plan(1, tA, tB, 1600, 1024, 4096)[0] == (15 if (tA, tB) == (0, 1) else 13)


@pytest.mark.parametrize("M,N,K,tile", [
    (8192, 4096, 1024, 14), (7936, 4096, 768, 14), (8192, 3584, 1024, 14), (8192, 3072, 1024, 11), (12288, 2816, 1024, 11), (4096, 8192, 512, 11),
    (13312, 2048, 1024, 11), (9472, 2048, 2816, 11),
    (8192, 32768, 512, 14), (6144, 4096, 4096, 14), (8192, 1024, 4096, 16), (6144, 1024, 4096, 11), (5120, 1024, 2048, 11), (5120, 1024, 1024, 12)])
def test_tiles_of_large_products(M, N, K, tile):
    """256x256 tiles (14) by how full their rounds are, not by whole rounds; 128x256 ones (16) for a nearly full round."""
    assert plan(1, 0, 1, M, N, K) == (tile, 1)


@pytest.mark.parametrize("M,N,K,products,tile", [
    (4096, 2048, 1024, 1, 11), (3072, 3072, 448, 1, 14), (3072, 3072, 384, 1, 11), (4096, 2304, 768, 1, 14),
    (12288, 2048, 512, 1, 11), (12288, 2048, 768, 1, 14), (12544, 2048, 512, 1, 14), (5120, 8192, 512, 1, 11), (5120, 8192, 768, 1, 14),
    (3072, 3072, 512, 2, 11), (2560, 4096, 512, 3, 14), (2048, 2048, 512, 4, 14), (9288, 832, 640, 1, 11), (12288, 576, 960, 1, 11),
    (14872, 576, 704, 1, 11), (57344, 128, 512, 1, 11), (98304, 128, 1024, 1, 11), (57344, 192, 512, 1, 14), (65536, 160, 4096, 1, 14),
    (65536, 128, 4096, 1, 14), (90000, 320, 512, 1, 11), (768, 64, 384, 512, 12), (768, 1024, 1024, 16, 14)])
def test_tiles_of_plain_products(M, N, K, products, tile):
    """A plain bf16 result takes 256x256 tiles from 144 of them on if 128x128 ones would not run in one round, and for one and a half
    rounds and more where 128x128 tiles would not fill whole rounds; the tiles of all products of a launch count, but not where
    more of them is past the edges than of 128x128 ones."""
    t, splits = ctypes.c_int(), ctypes.c_int()
    assert P.lib().ouro_op_gemm_plan_as(1, 0, 1, M, N, K, 0, 0, 0, products, ctypes.byref(t), ctypes.byref(splits)) == 0
    assert (t.value, splits.value) == (tile, 1)


@pytest.mark.parametrize("M,N,K,tile", [(2053, 570, 16, 1), (2053, 570, 17, 20), (1024, 512, 8, 20), (1056, 512, 8, 1), (1, 2082, 4, 20), (1, 1, 1, 20)])
def test_short_fp32_contractions(M, N, K, tile):
    for tA, tB in ((0, 0), (0, 1), (1, 0)):
        assert plan(0, tA, tB, M, N, K) == (tile, 1)


def test_reads_in_inline_assembly_wait_in_their_own_block():
    """The compiler takes the output registers of an asm block as written when the block ends: a load that is still under
    way then could be overtaken by whatever the compiler puts into them."""
    csrc = os.path.join(ROOT, "paper_1909_06695_amd", "csrc")
    reads = r"\b(ds_read|ds_load|global_load|buffer_load|flat_load|s_load)|_TEXT\b"      # ..._TEXT: lists of reads
    found = 0
    for name in sorted(os.listdir(csrc)):
        text = re.sub(r"//[^\n]*", "", open(os.path.join(csrc, name)).read())
        for block in re.findall(r"asm volatile\((.*?)\)\s*(?:;|\n)", text, flags=re.S):
            if re.search(reads, block):
                found += 1
                assert "s_waitcnt" in block, (name, block[:80])
    assert found >= 4


def group_plan(shapes, cleared, alone):
    n = len(shapes)
    ints = lambda i: (ctypes.c_int * n)(*[s[i] for s in shapes])
    tile, kchunk = ctypes.c_int(), ctypes.c_int()
    assert P.lib().ouro_op_gemm_group_plan(n, ints(0), ints(1), ints(2), cleared, alone, ctypes.byref(tile), ctypes.byref(kchunk)) == 0
    return tile.value, kchunk.value


def group_plan_over_every_range(shapes, cleared, alone):
    """The cost model of grouped weight gradients over every range length, with list scheduling slot by slot of time."""
    kmax = max((k + 63) // 64 * 64 for _, _, k in shapes)
    best = {}
    for kc in range(min(256, kmax), kmax + 1, 64):
        for bt, slots in ((128, 512), (256, 256)):
            part, adds = [], 0
            for m, w, k in shapes:
                s = -(-k // kc)
                n = -(-m // bt) * -(-w // bt) * s
                part.append((-(-(-(-k // s)) // 64), n))
                if s > 1 or not cleared:
                    adds += n * bt * bt
            wgs = sum(n for _, n in part)
            if alone:
                rate, fixed = (1.45, 6) if bt == 256 else (0.65 if wgs <= 256 else 0.82, 4)
                free, end = [(0.0, slots)], 0.0
                for r, left in sorted(part, key=lambda x: -x[0]):
                    while left:
                        free.sort()
                        at, have = free.pop(0)
                        take = min(left, have)
                        left -= take
                        if have > take:
                            free.append((at, have - take))
                        free.append((at + rate * r + fixed, take))
                        end = max(end, at + rate * r + fixed)
                cost = end + adds / (310e3 if bt == 256 else 400e3)
            else:
                one = 1.45 * (kc // 64) + 6 + adds / 310e3 if bt == 256 else 1.2 * (kc // 64 + 6)
                cost = 0.5 * one * (-(-wgs // slots) + wgs / slots)
            if cost < best.get(bt, (1e30,))[0] - 1e-9:
                best[bt] = (cost, kc)
    bt = 256 if best[256][0] < best[128][0] else 128
    return bt, best[bt][1]


LAYERS = [
    [(1024, 1024, 6144), (1024, 4096, 6144), (4096, 1024, 6144), (1024, 1024, 6144), (1024, 2048, 12288), (1024, 1024, 768)],
    [(448, 640, 4800), (640, 448, 4800), (448, 2112, 4800), (2112, 448, 4800), (448, 1280, 9600), (448, 640, 300)],
    [(64, 192, 8192), (64, 64, 8192), (64, 256, 8192), (256, 64, 8192)],
    [(512, 1536, 8192), (512, 512, 8192), (512, 2048, 8192), (2048, 512, 8192)],
    [(128, 384, 288), (128, 128, 288), (128, 256, 288), (256, 128, 288)],
    [(72, 40, 33)],
]


@pytest.mark.parametrize("alone", [0, 1])
@pytest.mark.parametrize("cleared", [0, 1])
def test_ranges_of_grouped_weight_gradients(cleared, alone):
    """The launcher looks at few range lengths; its choice is that of the whole search."""
    rng = random.Random(5)
    drawn = [[(rng.randrange(8, 2500, 8), rng.randrange(8, 2500, 8), rng.randrange(32, 9000)) for _ in range(rng.randrange(1, 7))] for _ in range(25)]
    for shapes in LAYERS + drawn:
        assert group_plan(shapes, cleared, alone) == group_plan_over_every_range(shapes, cleared, alone), shapes


def test_plan_of_grouped_weight_gradients_is_cheap():
    """Made on the host for every layer of every step: the best of many calls, as other work may run on this machine (86 and 61 us for
    the first two layers when every range was looked at)."""
    for shapes in LAYERS:
        n = len(shapes)
        args = [(ctypes.c_int * n)(*[s[i] for s in shapes]) for i in range(3)]
        tile, kchunk, f = ctypes.c_int(), ctypes.c_int(), P.lib().ouro_op_gemm_group_plan
        best = 1.0
        for _ in range(200):
            t = time.perf_counter()
            f(n, *args, 1, 1, ctypes.byref(tile), ctypes.byref(kchunk))
            best = min(best, time.perf_counter() - t)
        assert best < 45e-6, (shapes, best)


def test_waits_count_loads_by_name():
    """A wait that leaves younger memory operations under way counts them: by a constant of the kernel that issues them, not by a number
    that a merged or added operation would make wrong without a message."""
    csrc = os.path.join(ROOT, "paper_1909_06695_amd", "csrc")
    waits = [w for name in sorted(os.listdir(csrc)) if name.startswith("attention")
             for w in re.findall(r"fa_wait_vmcnt<([^;]*)>\(\);", open(os.path.join(csrc, name)).read())]
    assert len(waits) >= 6
    assert all(w == "0" or "LPT" in w for w in waits), waits


def test_lr_schedule_matches_the_oracle():
    """The library's host-side step-size function against the oracle's, over both phases and
    the boundaries (both fp64: agreement to rounding); bad arguments are refused."""
    from oracle import ouro_oracle as O
    for base, W, T, floor in [(2.5e-4, 5000, 200000, 0.0), (1e-3, 0, 1000, 1e-5), (0.1, 50, 51, 0.0), (3e-4, 500, 40000, 3e-6)]:
        for t in sorted({0, 1, W - 1 if W else 0, W, W + 1, (W + T) // 2, T - 1, T, T + 7, 12345 % (T + 1)}):
            got, ref = P.lr_schedule(base, W, T, t, floor), O.learning_rate(t, base, W, T, floor)
            assert abs(got - ref) <= 1e-15 + 1e-13 * abs(ref), (base, W, T, floor, t)
    for bad in [(1.0, 10, 10, 0, 0.0), (1.0, -1, 10, 0, 0.0), (1.0, 2, 10, -1, 0.0), (1.0, 2, 10, 0, 2.0), (1.0, 2, 10, 0, -0.1)]:
        with pytest.raises(P.OuroError):
            P.lr_schedule(bad[0], bad[1], bad[2], bad[3], bad[4])


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    """The stand-in for the HIP runtime, built; returns a function that runs a scenario of fake_hip_model.py on it."""
    here = os.path.join(ROOT, "tests")
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(here, "fake_hip.cpp")], check=True)

    def run(scenario):
        r = subprocess.run([sys.executable, os.path.join(here, "fake_hip_model.py"), so, scenario], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.endswith("passed\n"), r.stdout + r.stderr
    return run


def test_failed_step_leaves_no_partial_gradient(fake_hip):
    fake_hip("failed_step")


def test_steps_take_no_host_memory(fake_hip):
    fake_hip("steps_without_host_allocations")


def test_attention_of_many_short_streams_can_be_launched(fake_hip):
    fake_hip("attention_of_many_short_streams")


def test_updates_of_unaligned_matrices(fake_hip):
    fake_hip("updates_of_unaligned_matrices")


def test_bytes_of_a_timed_update(fake_hip):
    fake_hip("update_bytes")
