"""Failure handling of the library's host code, on the CPU: libwisv.so runs in a child process on a stand-in for the HIP
runtime (stub_hip.c: host memory, kernels logged instead of run) that fails where the test says."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes as C, sys
import numpy as np
sys.path.insert(0, ROOT)
from dataclasses import replace
from paper_2604_17701_amd import binding as B
from wisv_inputs import configs
stub = C.CDLL(STUB, mode=C.RTLD_GLOBAL)
stub.stub_log.restype = C.c_char_p
stub.stub_used.restype = C.c_size_t
stub.stub_limit.argtypes = [C.c_size_t]
lib = B.load_library()
SMALL = replace(configs.get(3).model, n_layers=2, d_model=256, n_heads=4, n_kv_heads=2, head_dim=128, d_ff=512, vocab=512, d_draft=64,
                d_head_hidden=64)


def create(model, max_batch, max_ctx, max_k):
    """a ctx on zero weights"""
    m = model
    cfg = B.make_config(m, max_batch, max_ctx, max_k)
    big = np.zeros(2 * max(m.vocab, 4 * m.d_ff, m.d_head_hidden, m.d_q) * max(m.d_model, m.d_ff, m.d_in, m.d_q), np.float32)
    w = B.wisv_weights()
    for name in ("embed", "lm_head", "final_norm", "head_w1", "head_b1", "head_w2", "head_b2"):
        setattr(w, name, big.ctypes.data)
    arr = (C.c_void_p * m.n_layers)(*[big.ctypes.data] * m.n_layers)
    for name in B._PER_LAYER:
        setattr(w, name, C.cast(arr, C.POINTER(C.c_void_p)))
    h, err = C.c_void_p(), C.create_string_buffer(512)
    rc = lib.wisv_ctx_create(C.byref(cfg), C.byref(w), C.byref(h), err, 512)
    assert rc == B.WISV_OK, err.value
    lib.wisv_set_state(h, 0, 0, 0)
    return h


def log():
    return [l for l in stub.stub_log().decode().split("\\n") if l]


def prefill(h, n):
    t = np.zeros(n, np.int32)
    return lib.wisv_prefill(h, 0, t.ctypes.data, n)


def state(h):
    a, b = C.c_int32(), C.c_int32()
    assert lib.wisv_get_state(h, 0, C.byref(a), C.byref(b)) == B.WISV_OK
    return a.value, b.value


def verify(h, model, batch, k):
    r = batch * k
    sid, toks, proto = np.arange(batch, dtype=np.int32), np.zeros(r, np.int32), np.zeros(batch, np.int32)
    hd, csi, tau = np.zeros((r, model.d_draft), np.float32), np.zeros((batch, model.d_csi), np.float32), np.zeros(batch, np.float32)
    out = [np.zeros(n, np.int32) for n in (batch, batch, r)]
    proto[:] = configs.PROTO_FH
    rin = B.wisv_round_in(batch, k, sid.ctypes.data, toks.ctypes.data, proto.ctypes.data, hd.ctypes.data, None, r, csi.ctypes.data,
                          tau.ctypes.data, 0)
    rout = B.wisv_round_out(*[o.ctypes.data for o in out], None, None, None)
    return lib.wisv_verify_round(h, C.byref(rin), C.byref(rout))


def ss_verify(h, model, batch, k):
    r = batch * k
    sid, toks = np.arange(batch, dtype=np.int32), np.zeros(r, np.int32)
    q, u, v = np.zeros((r, model.vocab), np.float32), np.zeros(r, np.float32), np.zeros(batch, np.float32)
    out = [np.zeros(n, np.int32) for n in (batch, batch, r)]
    sin = B.wisv_ss_in(batch, k, sid.ctypes.data, toks.ctypes.data, q.ctypes.data, u.ctypes.data, v.ctypes.data, 0)
    sout = B.wisv_ss_out(*[o.ctypes.data for o in out])
    return lib.wisv_ss_verify_round(h, C.byref(sin), C.byref(sout))

'''


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "stub_hip.so")
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-Werror", "-o", so, os.path.join(HERE, "stub_hip.c")])
    return so


def _run(stub, body):
    code = f"ROOT, STUB = {ROOT!r}, {stub!r}\n" + PRELUDE + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300, cwd=ROOT)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


def test_prompt_that_fails_half_way_leaves_the_slot_as_it_was(stub):
    """2500 tokens are three chunks; the copy of the third one's tokens fails after two chunks are enqueued, each of which
    moves the slot's length on the device.  The call must put the length back, wait for what it enqueued (the caller's
    tokens are still being read) and keep the host's bound on the length an upper bound, also when the wait itself fails."""
    _run(stub, """
    h = create(SMALL, 1, 2502, 4)
    stub.stub_log_clear()
    stub.stub_fail(2 + 1 + 3, 0, 0)              # two copies read the state, one writes the slot, then one per chunk
    assert prefill(h, 2500) == B.WISV_EHIP
    l = log()
    assert sum("k_set_pred_next" in x for x in l) == 3 and l[-1] == "sync", l[-5:]
    assert state(h) == (0, 0)
    assert prefill(h, 2500) == B.WISV_OK and state(h)[0] == 2500
    lib.wisv_set_state(h, 0, 0, 0)
    stub.stub_fail(2 + 1 + 3, 2, 0)              # the first wait belongs to the reading of the state
    assert prefill(h, 2500) == B.WISV_EHIP
    assert verify(h, SMALL, 1, 4) == B.WISV_ESTATE          # 2500 + 4 tokens may not fit
    assert state(h) == (0, 0) and verify(h, SMALL, 1, 4) == B.WISV_OK
    lib.wisv_destroy(h)
    """)


@pytest.mark.parametrize("call", ["verify", "ss_verify"])
@pytest.mark.parametrize("how", ["refused", "record"])
def test_failed_host_pointer_round_has_read_its_arguments(stub, call, how):
    """A host-pointer round that fails after its packed arguments were enqueued for copying must wait for that copy: the
    next call packs its own arguments into the same pinned memory.  Once because a product is not served (32 rows want
    more LDS than the runtime grants here), once because an event cannot be recorded."""
    _run(stub, f"""
    h = create(SMALL, 8, 64, 4)
    if {how == "refused"}:
        stub.stub_refuse_lds(1)
    else:
        stub.stub_fail(0, 0, {2 if how == "record" else 0})   # the record that ends the round
    stub.stub_log_clear()
    rc = {call}(h, SMALL, 8, 4)
    assert rc == (B.WISV_EUNSUPPORTED if {how == "refused"} else B.WISV_EHIP), rc
    l = log()
    assert any("k_unpack" in x for x in l) and l[-1] == "sync", l[-3:]
    stub.stub_refuse_lds(0)
    assert {call}(h, SMALL, 8, 4) == B.WISV_OK
    lib.wisv_destroy(h)
    """)


def test_prompt_buffers_are_not_part_of_the_context(stub):
    """What a ctx allocates depends on its rounds, not on how long its prompts may be; the first long prompt allocates its
    buffers, a device without room for them still ingests it (in chunks of half the rows, down to those of a round), and
    wisv_destroy gives everything back."""
    _run(stub, """
    def chunks(h, n):
        stub.stub_log_clear()
        lib.wisv_set_state(h, 0, 0, 0)
        assert prefill(h, n) == B.WISV_OK and state(h)[0] == n
        return sum("k_set_pred_next" in x for x in log())

    for model in (SMALL, configs.TINY):
        e = 2 if model.dtype == "bf16" else 4
        def grown(max_ctx):
            h = create(model, 1, max_ctx, 4)
            return h, stub.stub_used()
        h, small = grown(64)
        lib.wisv_destroy(h)
        assert stub.stub_used() == 0
        h, large = grown(1024)
        per_token = model.n_layers * 2 * model.n_kv_heads * model.head_dim * e + 2 * (model.head_dim // 2) * 4   # cache, rotary tables
        assert large - small == (1024 - 64) * per_token, (large - small, per_token)
        stub.stub_limit(large)
        assert chunks(h, 600) == 150 and stub.stub_used() == large       # no room at all: a round's four rows at a time
        stub.stub_limit(2 ** 62)
        assert chunks(h, 600) == 1
        full = stub.stub_used() - large
        assert chunks(h, 90) == 1 and stub.stub_used() - large == full   # kept, not grown
        lib.wisv_destroy(h)
        assert stub.stub_used() == 0
        h, large = grown(1024)
        stub.stub_limit(large + full - 1)
        assert chunks(h, 600) == 2 and stub.stub_used() < large + full   # half the rows
        lib.wisv_destroy(h)
        assert stub.stub_used() == 0
    """)


@pytest.mark.parametrize("call", ["verify", "ss_verify"])
def test_round_that_fails_after_its_commit_keeps_the_length_bound(stub, call):
    """The kernel that commits a round may have moved the stream's length when recording the round's last event fails: later
    rounds are checked against a bound that counts the whole block, until the state is read back."""
    _run(stub, f"""
    h = create(SMALL, 1, 64, 4)
    lib.wisv_set_state(h, 0, 60, 0)
    stub.stub_fail(0, 0, 2)
    assert {call}(h, SMALL, 1, 4) == B.WISV_EHIP
    assert {call}(h, SMALL, 1, 4) == B.WISV_ESTATE
    assert state(h) == (60, 0) and {call}(h, SMALL, 1, 4) == B.WISV_OK
    lib.wisv_destroy(h)
    """)
