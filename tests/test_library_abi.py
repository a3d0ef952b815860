"""Host-only checks of the C-ABI library: it loads, exports every symbol the header
declares, and rejects bad arguments before launching anything."""
import ctypes as C
import os
import re

import pytest

from paper_2510_19366_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_exports_match_header():
    hdr = open(os.path.join(ROOT, "include", "moe_prism.h")).read()
    declared = set(re.findall(r"MOE_PRISM_API\s+[\w\s\*]+?\b(moe_prism_\w+)\s*\(", hdr))
    assert declared == set(B.EXPORTS)
    lib = B.lib()
    for name in declared:
        assert hasattr(lib, name), name


def test_host_side_validation():
    lib = B.lib()
    n = C.c_size_t(0)
    ok = B.make_shape(64, 256, 8, 4, 128, 8, "f32")
    assert lib.moe_prism_workspace_bytes(C.byref(ok), C.byref(n)) == 0 and n.value > 0
    assert lib.moe_prism_workspace_bytes(C.byref(ok), None) == -1
    bad = [B.make_shape(64, 250, 8, 4, 128, 8, "f32"),        # d % 64
           B.make_shape(64, 256, 8, 4, 100, 8, "f32"),        # Is % 32
           B.make_shape(64, 256, 8, 4, 128, 33, "f32"),       # k_max > E
           B.make_shape(64, 256, 2048, 4, 128, 8, "f32")]     # E > 4096
    for s in bad:
        assert lib.moe_prism_workspace_bytes(C.byref(s), C.byref(n)) == -2
    neg = B.make_shape(-1, 256, 8, 4, 128, 8, "f32")
    assert lib.moe_prism_workspace_bytes(C.byref(neg), C.byref(n)) == -1
    # null pointers / missing workspace are refused on the host, nothing is launched
    assert lib.moe_prism_layer(C.byref(ok), None, None, None, None, None, None, None, None,
                               C.c_size_t(0), None) == -1
    assert lib.moe_prism_route(C.byref(ok), None, None, None, None, None, None, None, None,
                               C.c_size_t(0), None) == -1
    assert b"workspace" in lib.moe_prism_strerror(-3)
    # workspace grows with the pair capacity
    big = B.make_shape(128, 256, 8, 4, 128, 8, "f32")
    m = C.c_size_t(0)
    lib.moe_prism_workspace_bytes(C.byref(big), C.byref(m))
    assert m.value > n.value
    offs = B.moe_prism_layer_offsets(ok)
    assert all(v % 256 == 0 for v in offs.values()) and max(offs.values()) < n.value


@pytest.mark.parametrize("T,E,k_max,d,Is,dtype,env,path", [
    # narrow sub-experts: up to 64 tokens, and up to 24 possible rows; beyond, see below
    (64, 512, 32, 2048, 192, "bf16", "", "few"), (65, 512, 32, 2048, 192, "bf16", "", "few"),
    (159, 512, 32, 2048, 192, "bf16", "", "few"), (160, 512, 32, 2048, 192, "bf16", "", "few"),
    (384, 512, 32, 1024, 192, "bf16", "", "few"), (385, 512, 32, 1024, 192, "bf16", "", "fused"),
    (64, 4, 4, 2048, 192, "bf16", "", "few"), (65, 4, 4, 2048, 192, "bf16", "", "fused"),
    (192, 256, 32, 2048, 192, "bf16", "", "few"), (193, 256, 32, 2048, 192, "bf16", "", "fused"),
    (65, 256, 32, 2048, 192, "bf16", "split", "few"),
    (385, 256, 32, 2048, 192, "bf16", "split", "few"), (449, 256, 32, 2048, 192, "bf16", "split", "split"),
    (385, 256, 32, 192, 192, "bf16", "", "few"),     # d below the fused kernel's
    # others: up to 56 possible rows, any number for up to 64 tokens
    (597, 128, 12, 2048, 704, "bf16", "", "few"), (598, 128, 12, 2048, 704, "bf16", "", "split"),
    (64, 4, 4, 4096, 3584, "bf16", "", "few"), (65, 4, 4, 4096, 3584, "bf16", "", "split"),
    (8, 2, 1, 65536, 16384, "bf16", "", "split"),    # weights of a sub-expert beyond 32-bit offsets
    (8, 32, 8, 256, 128, "f32", "", "split")])
def test_ffn_path_is_the_rule_of_the_library(T, E, k_max, d, Is, dtype, env, path, monkeypatch):
    monkeypatch.setenv("MOE_PRISM_FFN", env)
    assert B.ffn_path(B.make_shape(T, d, E, 1, Is, k_max, dtype)) == path


@pytest.mark.parametrize("E,k_max,d,Is,most", [
    (512, 32, 2048, 192, 640), (512, 32, 4096, 192, 640),  # 40 possible rows for each, and 640 tokens
    (288, 32, 2048, 192, 360), (1024, 32, 2048, 192, 768), (1024, 80, 2048, 192, 512),  # 40; 24, more than 640 tokens; 40
    (512, 8, 2048, 192, 1536),                             # 24 possible rows are more than 640 tokens
    (512, 32, 2048, 128, 448), (288, 32, 2048, 128, 360),  # 448 tokens; 40 possible rows
    (512, 32, 1984, 192, 384), (512, 32, 2048, 64, 384), (512, 32, 256, 64, 384), (1024, 1, 1024, 128, 24576),  # 24
    (256, 16, 2048, 64, 384), (193, 12, 1024, 192, 386),   # 24, no more sub-experts than CUs
    (192, 12, 1024, 192, 896), (192, 12, 256, 64, 896), (8, 2, 2048, 128, 224)])  # 56, up to 3/4 as many as CUs
def test_ffn_path_of_narrow_sub_experts_up_to_the_last_batch_of_few_rows(E, k_max, d, Is, most, monkeypatch):
    # one range from the smallest batch on: nothing in between goes another way
    monkeypatch.setenv("MOE_PRISM_FFN", "")
    path = lambda T: B.ffn_path(B.make_shape(T, d, E, 1, Is, k_max, "bf16"))
    assert all(path(T) == "few" for T in range(1, most + 1))
    assert all(path(T) == "fused" for T in range(most + 1, most + 300))


def test_ffn_path_refuses_what_the_layer_refuses():
    out = C.c_int32(7)
    assert B.lib().moe_prism_ffn_path(C.byref(B.make_shape(64, 250, 8, 4, 128, 8, "bf16")), C.byref(out)) == -2
    assert B.lib().moe_prism_ffn_path(C.byref(B.make_shape(64, 256, 8, 4, 128, 8, "bf16")), None) == -1
    assert out.value == 7


def test_proxy_stage_that_would_overflow_the_tile_table_is_refused():
    # the proxy-gate stage cuts T*m pairs over N groups into the layer's tile table of
    # T*k_max/256 + E entries; a shape where they do not fit is refused on the host
    # (k_max = 2, m = 8: 2048 tiles needed, 1024 + 64 available)
    lib = B.lib()
    s = B.make_shape(65536, 256, 16, 4, 128, 2, "bf16")
    n = C.c_size_t(0)
    assert lib.moe_prism_workspace_bytes(C.byref(s), C.byref(n)) == 0
    dummy = (C.c_char * 256)()
    p = C.cast(dummy, C.c_void_p)
    rc = lib.moe_prism_route_proxy(C.byref(s), p, p, None, p, C.c_int32(8), C.c_int32(1),
                                   C.c_int32(32), p, p, p, p, p, C.c_size_t(n.value), None)
    assert rc == -2
    ok = B.make_shape(65536, 256, 16, 4, 128, 8, "bf16")          # m <= k_max always fits
    assert lib.moe_prism_workspace_bytes(C.byref(ok), C.byref(n)) == 0
    rc = lib.moe_prism_route_proxy(C.byref(ok), None, None, None, None, C.c_int32(8), C.c_int32(1),
                                   C.c_int32(32), None, None, None, None, None, C.c_size_t(0), None)
    assert rc == -1                                                 # passes the shape check, then null pointers
