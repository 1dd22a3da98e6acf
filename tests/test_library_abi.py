"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header
declares, and its host-only size arithmetic reproduces the byte accounting of
Sec. III-D.  No compute call is made."""
import ctypes as C
import os
import re

import pytest

from paper_2604_16864_amd import binding as hb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(hb._LIB_PATH):
        from paper_2604_16864_amd.build import build_lib
        build_lib(verbose=False)
    return hb.lib()


def test_exports_every_declared_symbol(L):
    hdr = "".join(open(os.path.join(ROOT, "include", f)).read() for f in sorted(os.listdir(os.path.join(ROOT, "include"))))
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(hs_[a-z_0-9]+)\s*\(", hdr))
    assert {"hs_compress_kv", "hs_prefill_attn", "hs_decode_attn", "hs_unpack_kv"} <= declared
    for name in declared:
        assert hasattr(L, name), name
    assert declared == set(hb.EXPORTS)


def test_size_arithmetic_matches_paper(L):
    sh = hb.make_shape(1, 32, 8, 32768)
    T = 32768 // 64
    c = hb.tile_counts(sh, hb.make_policy())
    assert c == [0, 0, T, 0, T]
    nb = hb.kv_bytes(sh, c)
    dense_total = 2 * 8 * 32768 * 128 * 2
    pools = nb[0] + nb[1] + nb[2] + nb[4] + nb[5] + nb[6]
    assert nb[1] + nb[2] == 8 * T * 9216
    assert round(dense_total / pools, 2) == 1.78                 # Sec. III-D: S_K = S_V = 1
    c = hb.tile_counts(sh, hb.make_policy(sparse_frac_k=0.5))
    nb = hb.kv_bytes(sh, c)
    pools = nb[0] + nb[1] + nb[2] + nb[4] + nb[5] + nb[6]
    assert round(dense_total / pools, 2) == 1.49                 # Sec. III-D: S_K = 0.5, S_V = 1
    c = hb.tile_counts(sh, hb.make_policy(skip_frac=0.75))
    assert c == [384, 0, 128, 0, 128]
    c = hb.tile_counts(sh, hb.make_policy(skip_frac=0.25, sparse_frac_k=0.0, sparse_frac_v=0.5))
    assert c == [128, 384, 0, 192, 192]


def test_protected_tiles_in_counts(L):
    sh = hb.make_shape(1, 32, 8, 32768)                          # T = 512
    # sink 64 tokens + local window 256 tokens dense (Sec. V-A), everything else 2:4
    c = hb.tile_counts(sh, hb.make_policy(dense_first_tiles=1, dense_last_tiles=4))
    assert c == [0, 5, 507, 5, 507]
    c = hb.tile_counts(sh, hb.make_policy(skip_frac=0.5, sparse_frac_v=0.5, dense_first_tiles=1, dense_last_tiles=4))
    assert c == [253, 5, 254, 5 + 127, 127]
    c = hb.tile_counts(sh, hb.make_policy(skip_frac=0.5, dense_first_tiles=400, dense_last_tiles=400))
    assert c == [0, 512, 0, 512, 0]
    cc = (C.c_int32 * 5)()
    assert L.hs_tile_counts(C.byref(sh), C.byref(hb.make_policy(dense_first_tiles=-1)), cc) == -1
    assert L.hs_tile_counts(C.byref(sh), C.byref(hb.make_policy(element_rule=2)), cc) == -1


def test_struct_layouts_match_the_header(tmp_path):
    """The ctypes mirrors have the size and field offsets the C compiler gives the header's structs."""
    fields = {"hs_shape": hb.HsShape, "hs_policy": hb.HsPolicy, "hs_kv": hb.HsKV}
    src = ['#include <stdio.h>', '#include <stddef.h>', '#include "hs.h"', 'int main(void) {']
    for cname, cls in fields.items():
        src.append(f'  printf("{cname} %zu", sizeof({cname}));')
        for f in cls._fields_:
            src.append(f'  printf(" %zu", offsetof({cname}, {f[0]}));')
        src.append('  printf("\\n");')
    consts = {"HS_BF16": hb.BF16, "HS_FP16": hb.FP16, "HS_RULE_MAGNITUDE": hb.RULE_MAGNITUDE,
              "HS_RULE_NONZERO": hb.RULE_NONZERO, "HS_MAP_F16": hb.MAP_F16}
    src.append('  printf("consts' + " %d" * len(consts) + '\\n", ' + ", ".join(consts) + ');')
    src += ['  return 0;', '}']
    c_file = tmp_path / "layout.c"
    c_file.write_text("\n".join(src))
    exe = tmp_path / "layout"
    import subprocess
    subprocess.run(["gcc", "-std=c99", "-I", os.path.join(ROOT, "include"), str(c_file), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    for line, (cname, cls) in zip(out, fields.items()):
        tok = line.split()
        assert tok[0] == cname
        assert int(tok[1]) == C.sizeof(cls), cname
        assert [int(x) for x in tok[2:]] == [getattr(cls, f[0]).offset for f in cls._fields_], cname
    assert [int(x) for x in out[len(fields)].split()[1:]] == list(consts.values())


def test_argument_errors(L):
    bad = hb.make_shape(1, 32, 8, 32768, D=64)
    c = (C.c_int32 * 5)()
    pol = hb.make_policy()
    assert L.hs_tile_counts(C.byref(bad), C.byref(pol), c) == -2
    odd = hb.make_shape(1, 32, 8, 1000)
    assert L.hs_tile_counts(C.byref(odd), C.byref(pol), c) == -2
    big_g = hb.make_shape(1, 32, 2, 1024)
    assert L.hs_tile_counts(C.byref(big_g), C.byref(pol), c) == -2
    ok = hb.make_shape(1, 4, 1, 1024)
    assert L.hs_tile_counts(C.byref(ok), C.byref(hb.make_policy(skip_frac=1.0)), c) == -1
    assert L.hs_tile_counts(C.byref(ok), C.byref(hb.make_policy(sparse_frac_k=1.5)), c) == -1
    assert L.hs_tile_counts(C.byref(ok), None, c) == -1
    # null buffers are rejected before anything is launched
    kv = hb.HsKV()
    assert L.hs_decode_attn(C.byref(ok), 0.0, 0, None, C.byref(kv), None, None, None, None) == -1
    assert L.hs_prefill_attn(C.byref(ok), 64, 0.0, 1, None, C.byref(kv), None, None, None, None) == -1
    assert L.hs_compress_kv(C.byref(ok), C.byref(pol), None, None, None, C.byref(kv), None, None) == -1
    assert L.hs_strerror(-2).decode().startswith("unsupported")
    # explicit states are device memory: the host cannot count them
    pol_s = hb.HsPolicy(0.0, 1.0, 1.0, 16, 16, None, None, 0, 0, 0)
    assert L.hs_tile_counts(C.byref(ok), C.byref(pol_s), c) == -2
    assert hb.workspace_bytes(ok, 2, 4) == 1 * 4 * 4 * 129 * 4
    assert hb.decode_auto_splits(ok) == 4


def test_prefill_workspace_rule(L):
    """Few queries on a long context ask for scratch, whole prompts and nearly empty caches do not."""
    def ranges(B, Hq, Hkv, L_, Lq, cap=None, causal=1, q_start=None):
        sh, kv, n = hb.make_shape(B, Hq, Hkv, L_), hb.HsKV(), C.c_size_t(0)
        kv.cap_sparse_k = L_ // 64 if cap is None else cap
        assert L.hs_prefill_workspace_bytes(C.byref(sh), Lq, L_ - Lq if q_start is None else q_start, causal, C.byref(kv), C.byref(n)) == 0
        assert n.value % (B * Hq * Lq * 129 * 4) == 0
        return n.value // (B * Hq * Lq * 129 * 4)
    assert ranges(1, 32, 8, 32768, 64) == 32 and ranges(1, 32, 8, 32768, 1024) == 2
    for L_ in (64, 256, 1024, 2048, 16384):
        assert ranges(1, 32, 8, L_, L_) == 0
    assert ranges(1, 32, 8, 32768, 64, cap=4) == 0 and ranges(1, 32, 8, 64, 64) == 0
    for B in (1, 3, 16):                              # bounded: at most 4096 workgroups of 66 KB
        for Lq in (64, 192, 2304, 4608, 32704):
            assert ranges(B, 32, 8, 65536, Lq) * B * 8 * (Lq // 32) <= 4096
    sh, n = hb.make_shape(1, 32, 8, 1024), C.c_size_t(0)
    kv = hb.HsKV()
    assert L.hs_prefill_workspace_bytes(C.byref(sh), 64, 1024, 1, C.byref(kv), C.byref(n)) == -1
    assert L.hs_prefill_workspace_bytes(C.byref(sh), 100, 0, 1, C.byref(kv), C.byref(n)) == -2
    assert L.hs_prefill_workspace_bytes(C.byref(sh), 64, 0, 1, None, C.byref(n)) == -1
    assert hb.workspace_bytes(sh, 1, 64) == 0         # the call without scratch needs none, as ever


def test_prefill_ranges_of_caches_whose_fill_the_host_does_not_know(L):
    """Pools with room for any state of every tile (states on the device) say nothing about how many tiles are kept:
    fewer ranges than for a full cache, none where three quarters skipped would not pay for them."""
    def ranges(B, T, Lq, caps, uniform=0):
        sh, kv, n = hb.make_shape(B, 32, 8, 64 * T), hb.HsKV(), C.c_size_t(0)
        kv.cap_dense_k, kv.cap_sparse_k, kv.cap_dense_v, kv.cap_sparse_v = caps
        kv.uniform = uniform
        assert L.hs_prefill_workspace_bytes(C.byref(sh), Lq, 64 * T - Lq, 1, C.byref(kv), C.byref(n)) == 0
        return n.value // (B * 32 * Lq * 129 * 4)
    for T in (64, 512):
        known = [((0, T, 0, T), 1), ((T // 4, T - T // 4, 0, T), 0)]      # the promise; shares of a fraction policy
        unknown = [((T, T, T, T), 0), ((0, T, 0, T), 0), ((T, 0, T, 0), 0), ((5, T, 5, T), 0)]
        B, Lq, full, some = (1, 64, 32, 16) if T == 512 else (2, 512, 2, 0)
        assert {ranges(B, T, Lq, *k) for k in known} == {full}
        assert {ranges(B, T, Lq, *k) for k in unknown} == {some}


def test_prefill_scratch_is_what_the_call_uses(L):
    """The binding asks for the workspace of the plan, and a call that gets exactly that much runs by the same plan."""
    def plan(B, Hq, Hkv, T, Lq, caps=None, causal=True, q_start=None):
        sh = hb.make_shape(B, Hq, Hkv, 64 * T)
        kv = hb.PackedKV(sh, caps or [0, 0, T, 0, T], "cpu")
        at = 64 * T - Lq if q_start is None else q_start
        slab, ranges, need = hb.prefill_plan(sh, Lq, at, kv, causal)
        one, most = B * Hq * Lq * 129 * 4, C.c_size_t(0)
        assert slab in (16, 32) and need == (ranges * one if ranges > 1 else 0)
        assert L.hs_prefill_workspace_bytes(C.byref(sh), Lq, at, int(causal), C.byref(kv.struct()), C.byref(most)) == 0 and need <= most.value
        assert hb.prefill_workspace_bytes(sh, Lq, at, kv, causal) == need
        for room in (need, max(need, one) + one - 1, most.value):
            assert hb.prefill_plan(sh, Lq, at, kv, causal, room) == (slab, ranges, need)
        assert hb.prefill_plan(sh, Lq, at, kv, causal, 0)[1:] == (1, 0)
        for n in range(2, ranges):
            assert hb.prefill_plan(sh, Lq, at, kv, causal, n * one)[1] <= n
        return slab, ranges
    assert plan(1, 32, 8, 512, 64) == (32, 32)
    assert plan(1, 32, 8, 32, 512) == (16, 1)                # a bound of two ranges, run in one
    assert plan(1, 32, 8, 128, 64) == (16, 8)                # a bound of 16
    for Hkv, G in ((8, 4), (1, 1), (3, 7), (2, 8)):
        for T, Lq in ((1, 64), (9, 128), (70, 64), (402, 192), (300, 2304), (2048, 64)):
            for B in (1, 2, 13):
                for caps in ([0, 0, T, 0, T], [0, T, 0, T, 0], [0, T, T, T, T], [0, T // 3, T - T // 3, 0, T], [T // 2, 0, T - T // 2, 0, T - T // 2]):
                    plan(B, G * Hkv, Hkv, T, Lq, caps)
    plan(2, 8, 2, 300, 128, causal=False, q_start=64 * 30 + 17)
    sh = hb.make_shape(1, 32, 8, 1024)
    kv = hb.PackedKV(sh, [0, 0, 16, 0, 16], "cpu")
    for bad in ((64, 1024), (0, 0), (100, 0), (64, -1)):
        with pytest.raises(hb.HsError):
            hb.prefill_plan(sh, *bad, kv)
    assert L.hs_prefill_plan(C.byref(sh), 64, 0, 1, None, 0, None, None, None) == -1
    assert L.hs_prefill_plan(C.byref(sh), 64, 0, 1, C.byref(kv.struct()), 0, None, None, None) == 0


def test_prefill_plan_with_its_teams(L):
    """The whole plan of a call, on both sides of the line for two teams of waves: one workgroup per compute unit and more, rows of
    few tiles, ranges, and a cache of mixed tiles."""
    def plan(L_, Lq, Hq=32, Hkv=8, B=1, caps=None, room=C.c_size_t(-1).value):
        sh = hb.make_shape(B, Hq, Hkv, L_)
        kv = hb.PackedKV(sh, caps or [0, 0, L_ // 64, 0, L_ // 64], "cpu")
        slab, ranges, need = hb.prefill_plan_teams(sh, Lq, L_ - Lq, kv, True, room)
        assert hb.prefill_plan(sh, Lq, L_ - Lq, kv, True, room) == (slab & ~hb.TWO_TEAMS, ranges, need)
        assert slab in (16, 32, 16 | hb.TWO_TEAMS) and (slab < 64 or ranges == 1)
        return slab, ranges
    two = 16 | hb.TWO_TEAMS
    assert plan(2048, 512) == (two, 1)                       # 256 workgroups, one per compute unit
    assert plan(2048, 576) == (16, 1)                        # 288
    assert plan(1024, 128) == (two, 1)                       # 64 workgroups of 16 tiles
    assert plan(256, 128) == (16, 1)                         # 64 of 4
    assert plan(1024, 1024) == (16, 1)                       # 512, a whole prompt
    assert plan(4096, 4096, Hq=4, Hkv=1) == (16, 3)          # 256 of up to 64 tiles
    assert plan(32768, 64) == (32, 32)                       # in ranges
    assert plan(32768, 64, room=0) == (two, 1)               # the same call without scratch
    assert plan(2048, 512, caps=[0, 16, 16, 0, 32]) == (two, 1)
    sh = hb.make_shape(1, 32, 8, 1024)
    kv = hb.PackedKV(sh, [0, 0, 16, 0, 16], "cpu")
    for bad in ((64, 1024), (0, 0), (100, 0), (64, -1)):
        with pytest.raises(hb.HsError):
            hb.prefill_plan_teams(sh, *bad, kv)
    assert L.hs_prefill_plan_teams(C.byref(sh), 64, 0, 1, None, 0, None, None, None) == -1
    assert L.hs_prefill_plan_teams(C.byref(sh), 64, 0, 1, C.byref(kv.struct()), 0, None, None, None) == 0


def test_current_stream_without_the_raw_handle(monkeypatch):
    """A torch without the two non-public functions gets the stream from the public object."""
    import torch

    class Stream:
        cuda_stream = 1234
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    for name in ("_raw_stream", "_current_device"):
        with monkeypatch.context() as m:
            m.setattr(hb, name, None)
            assert hb._stream() == 1234
    with monkeypatch.context() as m:
        m.setattr(hb, "_raw_stream", lambda dev: 100 + dev)
        m.setattr(hb, "_current_device", lambda: 3)
        assert hb._stream() == 103
