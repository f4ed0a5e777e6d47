"""The C ABI on the CPU: the library loads, exports every function that
include/dsv.h declares, and rejects bad host-known arguments with the
documented status codes before enqueueing anything (no GPU needed)."""
import ctypes
import os
import re

import pytest

import paper_2609_37532_amd as dsv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "dsv.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dsv_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_function():
    lib = dsv.load()
    names = declared_functions()
    assert len(names) >= 12
    for n in names:
        assert hasattr(lib, n), n


def test_no_bare_posix_names_exported():
    # a bare `accept` symbol would interpose accept(2) in the host process
    out = os.popen("nm -D --defined-only %s" % dsv.LIB_PATH).read()
    exported = {line.split()[-1] for line in out.splitlines() if " T " in line}
    assert "accept" not in exported and "verify_attn" not in exported
    assert all(n.startswith("dsv_") for n in exported if not n.startswith("_"))


def test_status_strings():
    expect = {0: "ok", -1: "null pointer argument", -2: "dimension out of range",
              -3: "unsupported configuration",
              -4: "workspace missing, misaligned or too small", -5: "HIP runtime error",
              -6: "exceeds the fixed scratch of the no-allocation entry point",
              7: "unknown status"}
    for code, text in expect.items():
        assert dsv.status_string(code) == text


def good_dims(**kw):
    d = dict(num_reqs=32, capacity=256, num_q_heads=32, num_kv_heads=8, head_dim=128,
             page_size=16, max_pages_per_req=514, num_pages=10000, max_kv_len=8208,
             scale=0.08838834764831845)
    d.update(kw)
    return dsv.AttnDims(**d)


@pytest.mark.parametrize("field,value,status", [
    ("num_reqs", 0, -2), ("capacity", 0, -2), ("num_q_heads", 30, -2),
    ("num_kv_heads", 0, -2), ("max_pages_per_req", 0, -2), ("num_pages", 0, -2),
    ("max_kv_len", 0, -2), ("max_kv_len", 514 * 16 + 1, -2), ("scale", 0.0, -2),
    ("scale", float("inf"), -2), ("page_size", 32, -3), ("head_dim", 96, -3),
    ("num_q_heads", 24, -3),  # G = 3 is not a power of two
])
def test_verify_attn_rejects_bad_dims(field, value, status):
    lib = dsv.load()
    d = good_dims(**{field: value})
    assert lib.dsv_verify_attn_workspace_bytes(ctypes.byref(d)) == 0
    fake = 1 << 20  # never dereferenced: validation fails first
    rc = lib.dsv_verify_attn(fake, fake, fake, fake, fake, fake, ctypes.byref(d), fake,
                             1 << 30, None)
    assert rc == status


def test_verify_attn_null_and_workspace_errors():
    lib = dsv.load()
    d = good_dims()
    need = lib.dsv_verify_attn_workspace_bytes(ctypes.byref(d))
    assert need > 0 and need % 256 == 0
    fake = 1 << 20
    assert lib.dsv_verify_attn(None, fake, fake, fake, fake, fake, ctypes.byref(d),
                               fake, need, None) == -1
    assert lib.dsv_verify_attn(fake, fake, fake, fake, fake, fake, None, fake, need,
                               None) == -1
    # too small, missing, misaligned workspace
    assert lib.dsv_verify_attn(fake, fake, fake, fake, fake, fake, ctypes.byref(d),
                               fake, need - 1, None) == -4
    assert lib.dsv_verify_attn(fake, fake, fake, fake, fake, fake, ctypes.byref(d),
                               None, need, None) == -4
    assert lib.dsv_verify_attn(fake, fake, fake, fake, fake, fake, ctypes.byref(d),
                               fake + 8, need, None) == -4
    # q, kv and out move in 16-byte vectors: misaligned views are refused
    for arg in (0, 2, 5):
        ptrs = [fake] * 6
        ptrs[arg] = fake + 2
        assert lib.dsv_verify_attn(*ptrs, ctypes.byref(d), fake, need, None) == -3, arg


def test_workspace_is_bounded_by_the_grid_not_the_context():
    # stream-K partials: at most two per workgroup of a grid capped at 1024,
    # so the workspace does not grow with the context length
    lib = dsv.load()
    ws = lambda **kw: lib.dsv_verify_attn_workspace_bytes(ctypes.byref(good_dims(**kw)))
    assert ws(max_kv_len=1024) == ws(max_kv_len=8208) > 0
    tiny = ws(num_reqs=1, num_kv_heads=1, num_q_heads=4, max_kv_len=64,
              max_pages_per_req=4)
    assert 0 < tiny < ws()
    # the flattened work must stay inside int32 indexing
    assert ws(num_reqs=65535, max_kv_len=8192) == 0


def test_int32_guard_counts_the_stream_k_lead_in():
    # The plan lays every segment after a lead-in of 192 virtual keys.  Here
    # the keys alone fit int32 indexing (256 * 65535 * 32 = 5.4e8 < 2^30),
    # but with the lead-in the work space is 256 * 65535 * 224 = 3.8e9 and
    # would overflow: the shape is refused before anything is enqueued.
    lib = dsv.load()
    d = good_dims(num_reqs=65535, num_kv_heads=256, num_q_heads=256, max_kv_len=32,
                  max_pages_per_req=2)
    assert lib.dsv_verify_attn_workspace_bytes(ctypes.byref(d)) == 0
    fake = 1 << 20
    assert lib.dsv_verify_attn(fake, fake, fake, fake, fake, fake, ctypes.byref(d), fake,
                               1 << 30, None) == -2
    # the boundary: the largest B that still fits with the lead-in is accepted
    seg = 32 + 192
    b_max = ((1 << 30) - 1) // (256 * seg)
    ok = good_dims(num_reqs=b_max, num_kv_heads=256, num_q_heads=256, max_kv_len=32,
                   max_pages_per_req=2)
    assert lib.dsv_verify_attn_workspace_bytes(ctypes.byref(ok)) > 0
    over = good_dims(num_reqs=b_max + 1, num_kv_heads=256, num_q_heads=256, max_kv_len=32,
                     max_pages_per_req=2)
    assert lib.dsv_verify_attn_workspace_bytes(ctypes.byref(over)) == 0


def test_accept_rejects_bad_arguments():
    lib = dsv.load()
    fake = 1 << 20
    need = lib.dsv_accept_workspace_bytes(256, 32, 151936)
    assert need > 0 and need % 256 == 0
    assert lib.dsv_accept_workspace_bytes(0, 32, 151936) == 0
    assert lib.dsv_accept_workspace_bytes(65536, 32, 151936) == 0
    # the counters sit at fixed offsets: a larger size never needs less space
    assert lib.dsv_accept_workspace_bytes(64, 8, 151936) <= need
    args = [fake, 1, fake, fake, fake, fake, 32, 256, 151936, fake, need, None]
    bad = list(args); bad[0] = None
    assert lib.dsv_accept(*bad) == -1
    bad = list(args); bad[1] = 7
    assert lib.dsv_accept(*bad) == -3
    bad = list(args); bad[6] = 0
    assert lib.dsv_accept(*bad) == -2
    bad = list(args); bad[8] = 0
    assert lib.dsv_accept(*bad) == -2
    bad = list(args); bad[10] = need - 1
    assert lib.dsv_accept(*bad) == -4
    bad = list(args); bad[9] = fake + 4
    assert lib.dsv_accept(*bad) == -4


def test_validate_and_graph_and_timing_argument_errors():
    lib = dsv.load()
    d = good_dims()
    fake = 1 << 20
    assert lib.dsv_validate_metadata(None, fake, fake, ctypes.byref(d), fake, None) == -1
    bad = good_dims(head_dim=80)
    assert lib.dsv_validate_metadata(fake, fake, fake, ctypes.byref(bad), fake, None) == -3
    assert lib.dsv_graph_capture_begin(None) == -1
    assert lib.dsv_graph_replay(None, None) == -1
    assert lib.dsv_graph_direct_launches(None) == -1
    assert lib.dsv_graph_destroy(None) == -1
    assert lib.dsv_timing_start(0) == -2
    assert lib.dsv_timing_stop(None, None) == -1


def test_binding_refuses_host_tensors():
    import torch
    q = torch.zeros(4, 2, 64, dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        dsv.verify_attn(q, torch.zeros(2, dtype=torch.int32),
                        torch.zeros(1, 2, 1, 1024, dtype=torch.bfloat16),
                        torch.zeros(1, 1, dtype=torch.int32),
                        torch.zeros(1, dtype=torch.int32), q.clone())


def test_dvl_rejects_bad_arguments():
    lib = dsv.load()
    fake = 1 << 20
    args = [fake] * 10 + [None, 32, 16, None]
    bad = list(args); bad[0] = None
    assert lib.dsv_dvl_allocate_pack(*bad) == -1
    bad = list(args); bad[9] = None
    assert lib.dsv_dvl_allocate_pack(*bad) == -1
    for n_bs in (0, dsv.DVL_MAX_REQS + 1):
        bad = list(args); bad[11] = n_bs
        assert lib.dsv_dvl_allocate_pack(*bad) == -2
    for w in (0, 1, 3, 15, 18):
        bad = list(args); bad[12] = w
        assert lib.dsv_dvl_allocate_pack(*bad) == -2


def test_accept_stochastic_rejects_bad_arguments():
    lib = dsv.load()
    fake = 1 << 20
    need = lib.dsv_accept_stochastic_workspace_bytes(256, 32, 151936)
    assert need > 0 and need % 256 == 0
    args = [fake, 1, fake, fake, fake, 1.0, fake, fake, 32, 256, 151936, fake, need, None]
    bad = list(args); bad[4] = None
    assert lib.dsv_accept_stochastic(*bad) == -1
    for t in (0.0, -1.0, float("inf"), float("nan"), 1e-45):
        bad = list(args); bad[5] = t
        assert lib.dsv_accept_stochastic(*bad) == -2, t
    bad = list(args); bad[1] = 3
    assert lib.dsv_accept_stochastic(*bad) == -3
    bad = list(args); bad[12] = need - 1
    assert lib.dsv_accept_stochastic(*bad) == -4


def test_predictor_rejects_bad_arguments():
    lib = dsv.load()
    fake = 1 << 20
    need = lib.dsv_predictor_workspace_bytes(32, 1735)
    assert need == 28 * 32 * 64 * 4 and lib.dsv_predictor_workspace_bytes(0, 1735) == 0
    args = [fake] * 7 + [32, 1735, 64, 15, fake, need, None]
    bad = list(args); bad[2] = None
    assert lib.dsv_predictor_forward(*bad) == -1
    bad = list(args); bad[7] = dsv.DVL_MAX_REQS + 1
    assert lib.dsv_predictor_forward(*bad) == -2
    bad = list(args); bad[10] = 0
    assert lib.dsv_predictor_forward(*bad) == -2
    bad = list(args); bad[9] = 32
    assert lib.dsv_predictor_forward(*bad) == -3
    bad = list(args); bad[12] = need - 1
    assert lib.dsv_predictor_forward(*bad) == -4


def test_read_probe_argument_errors():
    # every one of these is rejected on the host, before any launch
    lib = dsv.load()
    fake = 1 << 20
    assert lib.dsv_read_probe(None, 4, fake, 4, fake, 1, None) == -1
    assert lib.dsv_read_probe(fake, 4, None, 4, fake, 1, None) == -1
    assert lib.dsv_read_probe(fake, 4, fake, 4, None, 1, None) == -1
    assert lib.dsv_read_probe(fake, 0, fake, 4, fake, 1, None) == -2
    assert lib.dsv_read_probe(fake, 4, fake, 0, fake, 1, None) == -2
    assert lib.dsv_read_probe(fake, 4, fake, 4, fake, 0, None) == -2
    assert lib.dsv_read_probe(fake, 4, fake, 4, fake, 65536, None) == -2
    assert lib.dsv_read_probe(fake + 8, 4, fake, 4, fake, 1, None) == -3


def test_accept_noalloc_rejects_bad_arguments_before_any_device_call():
    # Every rejection below happens on the host, before the scratch address
    # is resolved or anything is enqueued (no GPU here).
    lib = dsv.load()
    fake = 1 << 20
    args = [fake, 1, fake, fake, fake, fake, 32, 256, 151936, None]
    bad = list(args); bad[3] = None
    assert lib.dsv_accept_noalloc(*bad) == -1
    bad = list(args); bad[1] = 7
    assert lib.dsv_accept_noalloc(*bad) == -3
    for i, v in ((6, 0), (7, 0), (7, 65536), (8, 0)):
        bad = list(args); bad[i] = v
        assert lib.dsv_accept_noalloc(*bad) == -2, (i, v)
    # the scratch limit: the need is the dsv_accept workspace size
    limit = 4 << 20
    assert lib.dsv_accept_workspace_bytes(256, 32, 151936) <= limit
    big = lib.dsv_accept_workspace_bytes(65535, 32, 262144)
    assert big > limit
    bad = list(args); bad[7] = 65535; bad[8] = 262144
    assert lib.dsv_accept_noalloc(*bad) == -6
    # the largest capacity that fits at a 151,936-token vocabulary (19 chunks)
    fits = max(c for c in range(27000, 28001)
               if lib.dsv_accept_workspace_bytes(c, 32, 151936) <= limit)
    assert lib.dsv_accept_workspace_bytes(fits + 1, 32, 151936) > limit
    assert fits >= 27000
