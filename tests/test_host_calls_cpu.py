"""What the library's host side queues, in which order and on which stream, on
the CPU: libspgemm.so bound to a stub of the HIP runtime (host/hip_stub.c) whose
kernels do nothing and whose header readings come from the test. Every scenario
runs in a process of its own (the stub has to be there before any HIP runtime).
"""
import ctypes as C
import importlib.util
import os
import re
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

# words of the device header (csrc/internal.h): columns per bin, errors, products
BIN_EMPTY, BIN_ESC0, BIN_SORT2, BIN_WSORT = 0, 1, 10, 12
W_ERR, W_CHUNKS, W_TOTAL_OP, W_HEAVY_PROD, W_HEAVY_WIN, W_NNZ = 36, 38, 40, 42, 44, 48
ERR_RETRY = 32
S1, S2, S3 = 0x1000, 0x2000, 0x3000


class Host:
    """The library on the stub, with one 4 x 4 problem's arrays."""

    def __init__(self, stub):
        self.stub = C.CDLL(stub, mode=C.RTLD_GLOBAL)
        self.stub.stub_log.restype = C.c_char_p
        spec = importlib.util.spec_from_file_location(
            "_lib", os.path.join(ROOT, "paper_2303_02471_amd", "_lib.py"))
        self.lib = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(self.lib)
        self.L = self.lib.lib()
        self.words = (C.c_uint32 * 4096).in_dll(self.stub, "stub_words")
        self.room = (C.c_double * 4096)()
        self.plan = C.c_void_p()
        self.nnz = C.c_int64()

    def at(self, i):
        return C.addressof(self.room) + 512 * i

    def header(self, bins, total_op, nnz, heavy=(0, 0), err=0):
        for i in range(64):
            self.words[i] = 0
        for b, n in bins.items():
            self.words[b] = n
        self.words[W_ERR], self.words[W_TOTAL_OP] = err, total_op
        self.words[W_HEAVY_PROD], self.words[W_HEAVY_WIN] = heavy
        self.words[W_NNZ] = nnz

    entries = 8

    def csc(self, base):
        return self.lib.Csc(4, 4, self.entries, self.at(base), self.at(base + 1), self.at(base + 2))

    def options(self, **kw):
        o = self.lib.Options()
        for k, v in kw.items():
            setattr(o, k, v)
        return C.byref(o)

    def multiply(self, stream=S1, dtype=1, opts=None, capacity=400):
        a, b = self.csc(0), self.csc(3)
        return self.L.spgemm_multiply(C.byref(a), C.byref(b), dtype, opts, stream,
                                      C.byref(self.plan), self.at(6), self.at(7), self.at(8),
                                      capacity, C.byref(self.nnz))

    def symbolic(self, stream=S1, dtype=1, opts=None):
        a, b = self.csc(0), self.csc(3)
        return self.L.spgemm_symbolic(C.byref(a), C.byref(b), dtype, opts, stream,
                                      C.byref(self.plan), self.at(6), C.byref(self.nnz))

    def numeric(self, stream):
        return self.L.spgemm_numeric(self.plan, self.at(2), self.at(5), self.at(7), self.at(8), stream)

    def backward(self, stream, da=True, db=True):
        return self.L.spgemm_backward(self.plan, self.at(2), self.at(5), self.at(7), self.at(8),
                                      self.at(9) if da else None, self.at(10) if db else None, stream)

    def batched(self, stream, values=None):
        """Size query of two problems, or (values: their value arrays) numeric."""
        a, b = self.csc(0), self.csc(3)
        if values:
            a.val, b.val = self.at(values), self.at(values + 1)
        As, Bs = (self.lib.Csc * 2)(a, a), (self.lib.Csc * 2)(b, b)
        two = (C.c_void_p * 2)
        nnz = (C.c_int64 * 2)()
        return self.L.spgemm_batched(2, As, Bs, 1, None, stream, C.byref(self.plan),
                                     two(self.at(6), self.at(7)), nnz,
                                     two(self.at(8), self.at(9)) if values else None,
                                     two(self.at(10), self.at(11)) if values else None)

    def log(self):
        lines = self.stub.stub_log().decode().split("\n")[:-1]
        self.stub.stub_clear()
        return lines

    def capture(self, stream):
        C.c_void_p.in_dll(self.stub, "stub_capturing").value = stream

    def fail(self, call, on, code):
        (C.c_char * 64).in_dll(self.stub, "stub_fail_call").value = call.encode()
        C.c_void_p.in_dll(self.stub, "stub_fail_on").value = on
        C.c_int.in_dll(self.stub, "stub_fail_code").value = code


def count(log, what):
    return sum(1 for x in log if re.search(what, x))


def first(log, what):
    return next(i for i, x in enumerate(log) if re.search(what, x))


SCENARIOS = {}


def scenario(f):
    SCENARIOS[f.__name__] = f
    return f


@scenario
def other_total_at_the_previous_positions_is_redone(h):
    """A product run at the previous structure's positions whose own total is
    another one: no kernel compares the columns that are empty now, so the
    totals decide, and the numeric phase runs again at the new positions."""
    h.header({BIN_EMPTY: 1, BIN_ESC0: 3}, 12, 9)
    assert h.multiply() == 0 and h.nnz.value == 9
    h.log()
    assert h.multiply() == 0 and h.nnz.value == 9
    same = h.log()
    assert count(same, "k_classify") == 1 and count(same, "k_acc_light") == 1
    h.header({BIN_EMPTY: 2, BIN_ESC0: 2}, 12, 6)
    assert h.multiply() == 0 and h.nnz.value == 6
    log = h.log()
    assert count(log, "k_classify") == 2, log
    # the last numeric launch comes after the scan that made the new pointers
    assert first(log[::-1], "k_acc_light") < first(log[::-1], "k_scan_small"), log


@scenario
def other_options_take_the_pass_with_the_read_back(h):
    """A planned launch runs on what the last call left; after a call with other
    options (or, in the product space, another value type) the sizes are read
    back and the scratch made first: two publications instead of one."""
    lib = h.lib
    default, radix = h.options(), h.options(flags=lib.SPGEMM_RADIX_ESC)
    hashed = h.options(flags=lib.SPGEMM_LANE_HASH)
    h.header({BIN_EMPTY: 2, BIN_SORT2: 2}, 3000, 100, heavy=(3000, 4))
    steps = ((default, 1, 2), (default, 1, 1), (radix, 1, 2), (radix, 1, 1), (default, 1, 2),
             (default, 1, 1), (default, 0, 1),  # (the direct scratch fits either type)
             (hashed, 0, 2), (hashed, 0, 1), (hashed, 1, 2), (hashed, 1, 1),
             (h.options(flags=lib.SPGEMM_LANE_HASH, t_split=-1), 1, 2), (default, 1, 2),
             (h.options(flags=lib.SPGEMM_ONE_STREAM), 1, 1))
    for i, (opts, dtype, passes) in enumerate(steps):
        assert h.multiply(dtype=dtype, opts=opts) == 0, i
        log = h.log()
        assert count(log, r"^publish") == passes, (i, log)


@scenario
def batch_table_waits_for_the_plans_earlier_work(h):
    """New value arrays on another stream: the copy over the problem table, which
    the last call's kernels read, is ordered behind them."""
    h.header({BIN_ESC0: 8}, 40, 15)
    h.words[W_NNZ + 2] = 15  # the second problem's
    assert h.batched(S1) == 0
    assert h.batched(S1, values=12) == 0
    h.log()
    assert h.batched(S2, values=14) == 0
    log = h.log()
    assert first(log, f"record .* stream {S1:#x}") < first(log, f"wait stream {S2:#x}") \
        < first(log, f"^copy .* stream {S2:#x}") < first(log, "k_acc_light"), log


@scenario
def batch_table_is_not_copied_inside_a_graph(h):
    """Arrays other than the last call's, on a stream under capture: refused
    (replays would copy from host memory that later calls write); the last
    call's arrays queue kernels only, and the plan goes on as before."""
    h.header({BIN_ESC0: 8}, 40, 15)
    h.words[W_NNZ + 2] = 15
    assert h.batched(S1) == 0
    assert h.batched(S1, values=12) == 0
    h.log()
    h.capture(S2)
    assert h.batched(S2, values=14) == 7
    log = h.log()
    assert not count(log, "^copy|^launch|^record"), log
    h.capture(None)
    assert h.batched(S1, values=12) == 0
    assert not count(h.log(), "^copy .* kind 2")
    h.capture(S2)
    assert h.batched(S2, values=12) == 0
    log = h.log()
    assert count(log, "^launch") and not count(log, "^copy|^sync|^await"), log
    h.capture(None)
    assert h.batched(S1, values=14) == 0 and count(h.log(), "^copy .* kind 1") == 1


@scenario
def host_memory_of_unfinished_work_is_not_pooled(h):
    """A plan destroyed while its stream cannot be waited for: the next plan takes
    other host memory. One destroyed in order hands its own on."""
    h.header({BIN_ESC0: 4}, 12, 9)

    def plan():
        h.plan = C.c_void_p()
        h.log()
        assert h.multiply() == 0
        return count(h.log(), "^hostalloc")

    assert plan() == 1
    h.L.spgemm_plan_destroy(h.plan)
    assert plan() == 0
    h.fail("hipStreamSynchronize", S1, 900)
    h.L.spgemm_plan_destroy(h.plan)
    h.fail("", None, 0)
    assert plan() == 1
    h.L.spgemm_plan_destroy(h.plan)


@scenario
def last_calls_stream_is_gone_or_under_capture(h):
    """The plan's last call ran on a stream that is destroyed since: the next
    numeric call on another one waits for the device and goes on. Or its last
    call was captured: nothing is recorded on the capturing stream."""
    h.header({BIN_ESC0: 4}, 12, 9)
    assert h.symbolic(S1) == 0
    assert h.numeric(S2) == 0
    h.log()
    h.fail("hipEventRecord", S2, 400)
    assert h.numeric(S1) == 0
    log = h.log()
    assert first(log, "^sync device") < first(log, "k_acc_light"), log
    h.fail("", None, 0)
    h.capture(S3)
    assert h.numeric(S3) == 0
    h.log()
    assert h.numeric(S1) == 0
    assert not count(h.log(), f"^record .* stream {S3:#x}")
    h.capture(None)


FORMS = {"one": ["k_gradI"], "two": ["k_grad_b", "k_grad_a"], "first pass": ["k_grad_b"],
         "apart": ["k_gradI", "k_grad_b"]}


def form(log):
    launched = [n for n in ("k_gradI", "k_grad_b", "k_grad_a") if count(log, n)]
    return next(k for k, v in FORMS.items() if v == launched)


@scenario
def gradients_take_the_faster_form(h):
    """The first call takes the two passes; once the longest lists are known, a
    few products on short lists take one launch, many or long lists two."""
    cases = (  # products, nnz(C), longest lists of dB and dA, form
        (40, 36, 8, 8, "one"),
        (40, 36, 900, 8, "two"),        # one long A column
        (40, 36, 8, 900, "two"),        # one long B row
        (3_000_000, 2_900_000, 8, 8, "two"),
        (3_000_000, 300_000, 8, 8, "one"))  # ten products on every entry of C
    h.entries = 400_000
    for products, nnz, zb, za, want in cases:
        h.header({BIN_ESC0: 4}, products, nnz)
        h.plan = C.c_void_p()
        assert h.symbolic(S1) == 0
        h.words[0], h.words[1] = zb, za
        h.log()
        assert h.backward(S1) == 0 and form(h.log()) == "two"
        assert h.backward(S1) == 0
        got = form(h.log())
        assert got == want, (products, zb, za, got)


@scenario
def captured_gradients_share_no_terms(h):
    """Many products: two passes through the plan's terms. A call under capture,
    whose replays may run beside other gradients of the plan, keeps the space it
    finds and the next call takes its own; without any, or after the fourth, dB
    keeps its pass, which writes no terms, and dA is formed in one launch."""
    h.entries, products = 400_000, 3_000_000
    h.header({BIN_ESC0: 4}, products, 2_900_000)
    terms = f"^alloc {8 * products} "
    assert h.symbolic(S1) == 0
    for i in range(6):
        h.log()
        assert h.backward(S1) == 0
        log = h.log()
        assert form(log) == "two" and count(log, terms) == (1 if i < 5 else 0), i
        h.capture(S2)
        assert h.backward(S2, da=False) == 0 and form(h.log()) == "first pass"
        for again in range(2):
            assert h.backward(S2) == 0
            log = h.log()
            assert form(log) == ("two" if i < 4 and again == 0 else "apart"), (i, again)
            assert not count(log, "^alloc|^sync|^await"), log
        assert h.backward(S2, db=False) == 0 and form(h.log()) == "one"
        h.capture(None)


@scenario
def terms_take_space_when_da_is_asked_for(h):
    """The space of one value per product: not for dB alone, nor under capture,
    and once."""
    h.entries, products = 400_000, 3_000_000
    h.header({BIN_ESC0: 4}, products, 2_900_000)
    assert h.symbolic(S1) == 0
    terms = f"^alloc {8 * products} "
    for da, stream, want in ((False, S1, 0), (False, S1, 0), (True, S2, 0), (True, S1, 1), (True, S1, 0),
                             (True, S2, 0), (True, S1, 1), (True, S1, 0)):
        h.capture(S2 if stream == S2 else None)
        h.log()
        assert h.backward(stream, da=da) == 0
        assert count(h.log(), terms) == want, (da, stream)
    h.capture(None)


@scenario
def numeric_tiles_alone_leave_room_in_the_caches(h):
    """The product space's numeric launch: unused LDS keeps tiles alone to four
    workgroups a compute unit (160 KB), not those beside chunks of large columns."""
    opts = h.options(flags=h.lib.SPGEMM_LANE_HASH)
    for bins, chunks in (({BIN_ESC0: 4}, 0), ({BIN_ESC0: 3, BIN_WSORT: 1}, 2)):
        h.plan = C.c_void_p()
        h.header(bins, 12000, 9000)
        h.words[W_CHUNKS] = chunks
        assert h.symbolic(S1, opts=opts) == 0
        h.log()
        assert h.numeric(S1) == 0
        lds = [int(re.search(r"lds (\d+)", x).group(1)) for x in h.log() if "k_numeric" in x]
        assert len(lds) == 1 and (lds[0] > 0) == (chunks == 0), (bins, lds)


@scenario
def pool_is_bounded_and_given_back(h):
    """Six plans end: the host memory of four is kept, the rest freed; four new
    plans take it, and spgemm_release_pool frees what is idle."""
    h.header({BIN_ESC0: 4}, 12, 9)

    def plans(n):
        made = []
        for _ in range(n):
            h.plan = C.c_void_p()
            assert h.multiply() == 0
            made.append(h.plan)
        return made, count(h.log(), "^hostalloc")

    def end(made):
        for p in made:
            h.L.spgemm_plan_destroy(p)
        return count(h.log(), "^hostfree")

    six, allocated = plans(6)
    assert allocated == 6 and end(six) == 2
    four, allocated = plans(4)
    assert allocated == 0 and end(four) == 0
    h.L.spgemm_release_pool()
    assert count(h.log(), "^hostfree") == 4
    one, allocated = plans(1)
    assert allocated == 1 and end(one) == 0


if __name__ != "__main__":
    import pytest

    @pytest.fixture(scope="module")
    def stub(tmp_path_factory):
        if shutil.which("gcc") is None:
            pytest.skip("needs gcc")
        if not os.path.exists(os.path.join(ROOT, "paper_2303_02471_amd", "libspgemm.so")):
            from paper_2303_02471_amd import build
            build.build()
        so = str(tmp_path_factory.mktemp("stub") / "libhip_stub.so")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so,
                        os.path.join(HERE, "host", "hip_stub.c")], check=True)
        return so

    @pytest.mark.parametrize("name", sorted(SCENARIOS))
    def test_host_calls(stub, name):
        r = subprocess.run([sys.executable, os.path.abspath(__file__), stub, name],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
else:
    SCENARIOS[sys.argv[2]](Host(sys.argv[1]))
