"""A model whose host side runs on the CPU over tests/fake_hip.cpp (no torch: its own HIP runtime would be found first).  Run as
a program: python fake_hip_model.py <stand-in library> <scenario>."""
import ctypes as C
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
E_STALE, E_HIP = -6, -7


class Config(C.Structure):
    _fields_ = ([(n, C.c_int32) for n in ("n_layer", "d_model", "n_head", "d_head", "d_ff", "vocab", "seq_len", "mem_len", "batch", "n_module")]
                + [("layers_per_module", C.POINTER(C.c_int32))] + [(n, C.c_int32) for n in ("rel_pos", "dtype", "optimizer")]
                + [(n, C.c_float) for n in ("beta1", "beta2", "eps")] + [("embed_warm_mode", C.c_int32), ("emb_scale", C.c_float),
                                                                         ("schedule", C.c_int32), ("dropout", C.c_float), ("seed", C.c_uint64)])


class Model:
    def __init__(self, fake, **kw):
        self.F = C.CDLL(fake, C.RTLD_GLOBAL)
        self.F.fake_name.restype = C.c_char_p
        self.F.fake_news.restype = C.c_long
        self.L = C.CDLL(os.path.join(ROOT, "paper_1909_06695_amd", "libouro.so"))
        c = dict(n_layer=3, d_model=32, n_head=2, d_head=16, d_ff=64, vocab=32, seq_len=8, mem_len=0, batch=2, n_module=3, rel_pos=0, dtype=0,
                 optimizer=0, beta1=0.9, beta2=0.999, eps=1e-8, emb_scale=1.0)
        c.update(kw)
        cfg, n = Config(**c), C.c_size_t()
        assert self.L.ouro_query_arena_bytes(C.byref(cfg), C.byref(n)) == 0
        self.buf = (C.c_char * (n.value + 256))()
        base = (C.addressof(self.buf) + 255) // 256 * 256
        self.h = C.c_void_p()
        assert self.L.ouro_create_model(C.byref(cfg), C.c_void_p(base), n, None, C.byref(self.h)) == 0
        self.K = c["n_module"]
        self.ids = C.c_void_p(C.addressof((C.c_int32 * (c["batch"] * c["seq_len"]))()))
        self.L.ouro_current_step.restype = C.c_int64

    def step(self, loss=True):
        x = C.c_float()
        return self.L.ouro_step(self.h, self.ids, self.ids, C.c_float(0.1), C.byref(x) if loss else None)

    def backward(self, k):
        return self.L.ouro_module_backward(self.h, k)

    def update(self, g):
        return self.L.ouro_delayed_update(self.h, g, C.c_float(0.1))

    def now(self):
        return self.L.ouro_current_step(self.h)

    def log(self, fn):
        """(result, [(kernel, first int of its arguments), ...]) of a call."""
        self.F.fake_reset()
        rc = fn()
        return rc, [(self.F.fake_name(i).decode(), self.F.fake_first_arg(i)) for i in range(self.F.fake_count())]

    def fail(self, launch, times=1):
        self.F.fake_fail(launch, times)


def sums(log):
    return [n for name, n in log if "sum_segments" in name]


def fills(log):
    return sum("fill_zero_kernel" in name for name, _ in log)


def failed_step(fake):
    """A step on one stream that fails at some launch: the modules whose backward pass had ended keep their whole gradient, or count
    as without one."""
    m = Model(fake)
    for _ in range(4):
        assert m.step() == 0
    rc, clean = m.log(m.step)
    assert rc == 0 and sums(clean) == [3]                  # the vector gradients of all three modules in one launch
    at = [i for i, (name, _) in enumerate(clean) if "sum_segments" in name][0]
    # in the backward pass of the last module: what the other two have added is summed on the way out
    m.fail(at - 3)
    rc, log = m.log(m.step)
    assert rc == E_HIP and sums(log) == [2], (rc, sums(log))
    tag = lambda k, depth: (m.L.ouro_debug_slot_tag(m.h, k, C.c_int64(5 % depth), C.byref(t)), t.value)[1]
    t = C.c_int64()
    # iteration 5: modules 3 and 2 have theirs; the cleared slots of module 1 (of iteration 2 before) and of dV_i hold nothing
    assert (tag(3, 1), tag(2, 2), tag(1, 3), tag(0, 3)) == (5, 5, -1, -1)
    rc, log = m.log(lambda: m.backward(1))
    assert rc == 0 and sums(log) == [1]
    extra = fills(log)
    assert all(m.update(g) == 0 for g in range(4)) and m.now() == 6
    # the copies that the failed module left were cleared first: one fill more than without a failure
    assert all(m.L.ouro_module_forward(m.h, k, m.ids, m.ids) == 0 for k in (1, 2, 3)) and m.backward(3) == 0 and m.backward(2) == 0
    rc, log = m.log(lambda: m.backward(1))
    assert rc == 0 and fills(log) == extra - 1
    assert all(m.update(g) == 0 for g in range(4)) and m.now() == 7
    # nothing can be launched any more, then everything again: the top module's gradient is refused (the others' are older ones)
    m.fail(at - 3, 1000)
    rc, log = m.log(m.step)
    assert rc == E_HIP and sums(log) == []
    m.fail(-1)
    assert m.backward(1) == 0
    assert m.update(3) == E_STALE
    # the launch of the sums itself
    m = Model(fake)
    for _ in range(4):
        assert m.step() == 0
    m.fail(at)
    assert m.step() == E_HIP
    assert m.update(3) == E_STALE


def steps_without_host_allocations(fake):
    """Nothing throws across the C boundary: a step, which every caller makes again and again, takes no host memory."""
    for kw in (dict(), dict(n_module=1), dict(dtype=1, d_model=128, d_head=64, d_ff=128, optimizer=1),
               dict(dtype=1, d_model=128, d_head=64, d_ff=128, seq_len=16, mem_len=24, rel_pos=1), dict(schedule=1, dropout=0.1)):
        m = Model(fake, **kw)
        for on in (0, 1):
            assert m.L.ouro_debug_set_overlap(m.h, on) == 0
            m.F.fake_news(1)
            for _ in range(5):
                assert m.step() == 0
            assert m.F.fake_news(0) == 0, (kw, on)


def attention_of_many_short_streams(fake):
    """fp32 attention over 65535 streams of one query and 129 heads: no axis of a grid has 2^32 threads (launches fail there)."""
    m = Model(fake)
    B, H, x = 65535, 129, C.c_void_p(256)
    ldv = 2 * H
    fwd = (None, 0, B, H, 1, 1, 2, 0, C.c_float(1.0), x, ldv, x, ldv, x, ldv, x, ldv, x)
    rc, log = m.log(lambda: m.L.ouro_op_attention_fwd(*fwd, 0, None, None, None, 0, 0))
    assert rc == 0 and len(log) == 1
    rc, log = m.log(lambda: m.L.ouro_op_attention_bwd(*fwd, x, ldv, x, ldv, x, ldv, x, ldv, 0, None, None, None, 0, None, None, None, x, 0))
    assert rc == 0 and len(log) == 1 and "af_bwd" in log[0][0], (rc, log)


def updates_of_unaligned_matrices(fake):
    """Matrices with rows off 16 bytes go to the plain update and the transposing kernel where they are large, the rest to the tile-wise
    one; all of it to that where the rows are aligned."""
    for d_head, vocab, want in ((65, 2000, {"groups": 1}), (65, 3000, {"groups": 1, "plain": 1, "transpose": 1}), (66, 3000, {"groups": 1}),
                                (127, 100, {"groups": 1, "plain": 3, "transpose": 3})):
        m = Model(fake, dtype=1, d_head=d_head, d_model=2 * d_head, d_ff=2 * d_head, vocab=vocab, optimizer=1)
        assert m.step() == 0
        rc, log = m.log(m.step)
        count = lambda what: sum(what in name for name, _ in log)
        got = {"groups": count("update_groups_kernel"), "plain": count("13update_kernel"), "transpose": count("transpose_table")}
        assert rc == 0 and {k: v for k, v in got.items() if v} == want, (d_head, vocab, got)


def update_bytes(fake):
    """The bytes that the update's timing counts: both bf16 copies where its launch writes both."""
    for dtype, aligned in ((0, True), (1, True), (1, False)):
        d, F, V = (128, 128, 3000) if aligned else (130, 130, 3001)
        m = Model(fake, dtype=dtype, d_head=d // 2, d_model=d, d_ff=F, vocab=V, optimizer=1)
        for _ in range(4):
            assert m.step() == 0
        m.L.ouro_debug_timing_enable(m.h, 1)
        assert m.step() == 0
        ms, n, work = C.c_double(), C.c_int64(), C.c_double()
        assert m.L.ouro_debug_timing_read(m.h, 1, C.byref(ms), C.byref(n), C.byref(work)) == 0
        mats = 4 * d * d + 2 * d * F
        layer = mats + 5 * d + F
        per = 4 + 8 + 16 + 2 * dtype
        want = per * 3 * layer + (per + 4) * V * d             # V takes two gradients
        want += dtype * 2 * (3 * mats + (V * d if aligned else 0))
        assert n.value == 1 and work.value == want, (dtype, aligned, work.value, want)


if __name__ == "__main__":
    globals()[sys.argv[2]](sys.argv[1])
    print("passed")
