"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same
seeded inputs.  Packed values, metadata, pools and maps: bit-exact.  Attention
outputs: max|d| <= 1e-2 * max|ref| and mean|d| / mean|ref| <= 2e-3."""
import numpy as np
import pytest
import torch

from oracle import hs_layout as hl
from oracle import hs_oracle as orc
from paper_2604_16864_amd import binding as hb
from paper_2604_16864_amd import workloads as wl

pytestmark = pytest.mark.gpu

MAX_TOL, MEAN_TOL = 1e-2, 2e-3


def _dev(bits, dtype="bf16"):
    return hb.bits_to_bf16_tensor(bits, "cuda", torch.float16 if dtype == "fp16" else torch.bfloat16)


def _f32(t):
    return t.float().cpu().numpy().astype(np.float64)


def assert_close(out, ref, what):
    out = np.asarray(out, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert np.isfinite(out).all(), what
    err = np.abs(out - ref)
    mx, mean = err.max() / max(np.abs(ref).max(), 1e-30), err.mean() / max(np.abs(ref).mean(), 1e-30)
    print(f"[{what}] max rel {mx:.3e} mean rel {mean:.3e}", flush=True)
    assert mx <= MAX_TOL, (what, mx)
    assert mean <= MEAN_TOL, (what, mean)


def assert_lse_close(lse, ref, what):
    lse = np.asarray(lse, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    inf = np.isneginf(ref)
    assert (np.isneginf(lse) == inf).all(), what
    assert np.allclose(lse[~inf], ref[~inf], rtol=1e-4, atol=1e-4), (what, np.abs(lse[~inf] - ref[~inf]).max())


def _prefill(sh, Q, kv, causal=True, scale=0.0, q_start=None):
    """hb.prefill_attn, whose result the test holds against the oracle, after the kernels that the library did not choose for so
    small a call (slabs of 16 and of 32 queries, in one range and in two, and two teams of waves) have been held against it: as close
    to it as each has to be to the oracle, head by head."""
    O, LSE = hb.prefill_attn(sh, Q, kv, causal=causal, scale=scale, q_start=q_start)
    ref, lref = _f32(O), LSE.cpu().numpy()
    assert np.isfinite(ref).all()
    for slab, n in ((16, 1), (16, 2), (32, 1), (32, 2), (16 | hb.TWO_TEAMS, 1)):
        Os, Ls = hb.prefill_attn_planned(sh, Q, kv, slab, n, causal=causal, scale=scale, q_start=q_start)
        err = np.abs(_f32(Os) - ref)
        assert (err.max((2, 3)) <= MAX_TOL * np.abs(ref).max((2, 3))).all(), (slab, n)
        assert (err.mean((2, 3)) <= MEAN_TOL * np.abs(ref).mean((2, 3))).all(), (slab, n)
        assert_lse_close(Ls.cpu().numpy(), lref, (slab, n))
    return O, LSE


def compress_both(B, Hq, Hkv, L, K, V, dtype="bf16", **pol):
    sh = hb.make_shape(B, Hq, Hkv, L, dtype=hb.FP16 if dtype == "fp16" else hb.BF16)
    lib_pol = dict(pol)
    if "element_rule" in lib_pol:
        lib_pol["element_rule"] = {"magnitude": hb.RULE_MAGNITUDE, "nonzero": hb.RULE_NONZERO}[lib_pol["element_rule"]]
    policy = hb.make_policy(**lib_pol)
    kv = hb.compress_kv(sh, policy, _dev(K, dtype), _dev(V, dtype))
    torch.cuda.synchronize()
    hb.check_state_flag(policy)          # explicit states: nothing left out, every pair valid
    pk, pv, info = orc.compress_kv(K, V, Bt=64, dtype=dtype, **pol)
    return sh, kv, pk, pv, info


def lib_maps(k_map, v_map):
    """The library's map arrays as (signed index map of K, signed index map of V, encoding flag of V):
    a v_map entry of a bf16 cache may carry HS_MAP_F16 in its magnitude, which is not part of the
    paper's signed index map (Sec. III-B) and is compared on its own."""
    km = k_map.cpu().numpy()
    vm = v_map.cpu().numpy().astype(np.int64)
    mag = np.abs(vm)
    assert not ((np.abs(km.astype(np.int64)) & hb.MAP_F16) != 0).any()
    return km, (np.sign(vm) * (mag & ~hb.MAP_F16)).astype(np.int32), (mag & hb.MAP_F16) != 0


def assert_maps_equal(kv, pk, pv, sel=None, osel=None):
    """sel / osel: index into the library's / the oracle's [B, Hkv, T] arrays (default: everything)."""
    km, vm, flag = lib_maps(kv.k_map if sel is None else kv.k_map[sel], kv.v_map if sel is None else kv.v_map[sel])
    o = (lambda a: a) if osel is None else (lambda a: a[osel])
    assert (km == o(pk.map)).all() and (vm == o(pv.map)).all(), "signed index maps"
    assert (flag == o(pv.f16)).all(), "fp16-encoding predicate of the V tiles"


def check_packed_bit_exact(sh, kv, pk, pv):
    assert_maps_equal(kv, pk, pv)
    B, H = sh.B, sh.Hkv
    for name, p, dense, nnz, meta, cd, cs in (("k", pk, kv.k_dense, kv.k_nnz, kv.k_meta, kv.counts[1], kv.counts[2]),
                                               ("v", pv, kv.v_dense, kv.v_nnz, kv.v_meta, kv.counts[3], kv.counts[4])):
        ph = hl.physical_pools(p)
        for b in range(B):
            for h in range(H):
                nd, ns = int(ph["n_dense"][b, h]), int(ph["n_sparse"][b, h])
                assert nd <= cd and ns <= cs
                if nd:
                    got = dense.cpu().numpy().reshape(B, H, cd, 16384)[b, h, :nd]
                    assert (got == ph["dense"][b, h, :nd]).all(), (name, "dense", b, h)
                if ns:
                    got = nnz.cpu().numpy().reshape(B, H, cs, 8192)[b, h, :ns]
                    assert (got == ph["nnz"][b, h, :ns]).all(), (name, "nnz", b, h)
                    got = meta.cpu().numpy().reshape(B, H, cs, 1024)[b, h, :ns]
                    assert (got == ph["meta"][b, h, :ns]).all(), (name, "meta", b, h)
    Ku, Vu = hb.unpack_kv(sh, kv)
    torch.cuda.synchronize()
    assert (hb.bf16_tensor_to_bits(Ku) == orc.unpack_tensor(pk)).all()
    assert (hb.bf16_tensor_to_bits(Vu) == orc.unpack_tensor(pv)).all()


def _mixed_states(B, Hkv, T, seed, p_skip=0.2):
    rng = np.random.default_rng(seed)
    sk = rng.choice([1, 2], size=(B, Hkv, T)).astype(np.int8)
    sv = rng.choice([1, 2], size=(B, Hkv, T)).astype(np.int8)
    skip = rng.random((B, Hkv, T)) < p_skip
    sk[skip] = 0
    sv[skip] = 0
    return sk, sv


# ------------------------------------------------------------------ compress
def test_compress_cfg0_bit_exact():
    c, Q, K, V = wl.make_config("cfg0_decode_small")
    # plant ties, zeros, negative zeros and an all-zero group
    K[0, 0, 5, :8] = wl.f32_to_bf16_bits(np.array([1, 1, -1, 1, 0, -0.0, 0, 0], dtype=np.float32))
    V[0, 0, 8:12, 7] = wl.f32_to_bf16_bits(np.array([2, -2, 2, -2], dtype=np.float32))
    sh, kv, pk, pv, _ = compress_both(c["B"], c["Hq"], c["Hkv"], c["L"], K, V)
    check_packed_bit_exact(sh, kv, pk, pv)
    assert kv.nbytes == pk.nbytes() + pv.nbytes()


def test_compress_explicit_mixed_states_bit_exact():
    B, Hq, Hkv, L = 2, 8, 2, 64 * 11
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 64, seed=21)
    sk, sv = _mixed_states(B, Hkv, L // 64, seed=22)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, state_k=sk, state_v=sv)
    check_packed_bit_exact(sh, kv, pk, pv)


def test_compress_strided_input():
    """K, V as slices of a wider buffer (token stride 256 elements)."""
    B, Hq, Hkv, L = 1, 4, 2, 256
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 64, seed=23)
    sh = hb.make_shape(B, Hq, Hkv, L)
    wide_k = torch.zeros((B, Hkv, L, 256), dtype=torch.bfloat16, device="cuda")
    wide_v = torch.zeros_like(wide_k)
    wide_k[..., :128] = _dev(K)
    wide_v[..., :128] = _dev(V)
    kv = hb.compress_kv(sh, hb.make_policy(), wide_k[..., :128], wide_v[..., :128])
    pk, pv, _ = orc.compress_kv(K, V)
    check_packed_bit_exact(sh, kv, pk, pv)


@pytest.mark.parametrize("skip,sfk,sfv", [(0.25, 1.0, 1.0), (0.5, 1.0, 1.0), (0.75, 1.0, 1.0), (0.25, 0.5, 1.0),
                                          (0.0, 0.3, 0.7), (0.5, 0.0, 0.0)])
def test_compress_policy_ranking(skip, sfk, sfv):
    B, Hq, Hkv, L = 2, 8, 2, 64 * 40
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 64, seed=31)
    # an exact tie in energy and in loss: two identical tiles
    K[0, 0, 64 * 9:64 * 10] = K[0, 0, 64 * 3:64 * 4]
    V[0, 0, 64 * 9:64 * 10] = V[0, 0, 64 * 3:64 * 4]
    sh, kv, pk, pv, info = compress_both(B, Hq, Hkv, L, K, V, skip_frac=skip, sparse_frac_k=sfk, sparse_frac_v=sfv)
    # fp64 sums in a different order: scores agree to ~1e-15; the cut must not sit on a
    # near-tie other than the planted exact one for the maps to be unique
    for key in ("energy", "loss_k", "loss_v"):
        s = np.sort(info[key], axis=-1)
        gaps = np.diff(s, axis=-1) / s[..., 1:]
        assert ((gaps > 1e-12) | (gaps == 0)).all()
    check_packed_bit_exact(sh, kv, pk, pv)


@pytest.mark.parametrize("skip,sfk,sfv,first,last", [(0.0, 1.0, 1.0, 1, 2), (0.5, 1.0, 1.0, 1, 4), (0.25, 0.5, 0.3, 2, 3),
                                                     (0.0, 1.0, 0.0, 3, 0), (0.5, 1.0, 1.0, 30, 30)])
def test_compress_protected_end_tiles(skip, sfk, sfv, first, last):
    """Sink / local-window tiles stay dense (both the host-built map path and the ranked one);
    the all-zero end tiles would be the first skipped if they took part in the ranking."""
    B, Hq, Hkv, L = 2, 8, 2, 64 * 40
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=33)
    K[0, 0, :64] = 0
    V[0, 0, :64] = 0
    K[1, 1, -64:] = 0
    V[1, 1, -64:] = 0
    pol = dict(skip_frac=skip, sparse_frac_k=sfk, sparse_frac_v=sfv, dense_first_tiles=first, dense_last_tiles=last)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, **pol)
    assert (pk.map[:, :, :min(first, 40)] > 0).all() and (pv.map[:, :, 40 - min(last, 40 - min(first, 40)):] > 0).all()
    check_packed_bit_exact(sh, kv, pk, pv)
    q = Q[:, :, 0, :].copy()
    O, LSE = hb.decode_attn(sh, _dev(q), kv)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, pk, pv)
    assert_close(_f32(O), Or, f"decode protected tiles {pol}")
    assert_lse_close(LSE.cpu().numpy(), Lr, "decode protected tiles lse")


@pytest.mark.parametrize("sfk,sfv", [(1.0, 1.0), (1.0, 0.0), (0.0, 1.0)])
@pytest.mark.parametrize("T,first,last", [(6, 1, 4), (6, 0, 1), (6, 3, 0), (5, 1, 4), (4, 2, 9), (1, 0, 1), (7, 0, 0)])
def test_compress_protected_end_tiles_without_ranking(T, first, last, sfk, sfv):
    """Entries that follow from the tile's index: sinks and windows of every size, up to all of the row."""
    Q, K, V = wl.make_qkv(2, 2, 2, 64 * T, 128, 1, seed=40 + T)
    sh, kv, pk, pv, _ = compress_both(2, 2, 2, 64 * T, K, V, sparse_frac_k=sfk, sparse_frac_v=sfv, dense_first_tiles=first,
                                      dense_last_tiles=last)
    check_packed_bit_exact(sh, kv, pk, pv)


def test_compress_nonzero_rule_premasked_input():
    """Generic compressor (Sec. IV-B): K, V arrive with an arbitrary 2:4 element mask applied
    (zeros at pruned places); under the non-zero rule the packed form decodes to the input."""
    B, Hq, Hkv, L = 1, 4, 2, 64 * 6
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=35)
    rng = np.random.default_rng(36)
    K[K == 0] = 0x3F80
    V[V == 0] = 0x3F80
    pairs = np.array([[1, 1, 0, 0], [1, 0, 1, 0], [1, 0, 0, 1], [0, 1, 1, 0], [0, 1, 0, 1], [0, 0, 1, 1]], dtype=bool)
    mk = pairs[rng.integers(0, 6, size=(B, Hkv, L, 32))].reshape(B, Hkv, L, 128)
    mv = pairs[rng.integers(0, 6, size=(B, Hkv, L // 4, 128))].transpose(0, 1, 2, 4, 3).reshape(B, Hkv, L, 128)
    Km, Vm = np.where(mk, K, 0).astype(np.uint16), np.where(mv, V, 0).astype(np.uint16)
    Km[0, 0, 7, 0:8] = [0, 0x4000, 0, 0, 0, 0, 0, 0]        # one survivor; an empty group
    Vm[0, 1, 8:12, 5] = [0x8000, 0, 0xC000, 0x4000]         # a negative zero counts as pruned
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, Km, Vm, element_rule="nonzero", skip_frac=0.2, sparse_frac_k=0.75)
    check_packed_bit_exact(sh, kv, pk, pv)
    Ku, Vu = hb.unpack_kv(sh, kv)
    kept = np.repeat(pk.map != 0, 64, axis=-1)[..., None]
    Vw = Vm.copy()
    Vw[0, 1, 8, 5] = 0
    assert (hb.bf16_tensor_to_bits(Ku) == np.where(kept, Km, 0)).all()
    assert (hb.bf16_tensor_to_bits(Vu) == np.where(kept, Vw, 0)).all()


# ------------------------------------------------------------------ decode
def _decode_case(B, Hq, Hkv, L, seed, n_splits=0, k_outliers=False, **pol):
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=seed, k_outliers=k_outliers)
    q = Q[:, :, 0, :].copy()
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, **pol)
    O, LSE = hb.decode_attn(sh, _dev(q), kv, n_splits=n_splits)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, pk, pv)
    return _f32(O), LSE.cpu().numpy(), Or, Lr


def test_decode_cfg0_full():
    c, q, K, V = wl.make_config("cfg0_decode_small")
    sh, kv, pk, pv, _ = compress_both(c["B"], c["Hq"], c["Hkv"], c["L"], K, V)
    Or, Lr = orc.attention_decode(q, pk, pv)
    for ns in (0, 1, 2, 7, 32):
        O, LSE = hb.decode_attn(sh, _dev(q), kv, n_splits=ns)
        torch.cuda.synchronize()
        assert_close(_f32(O), Or, f"decode cfg0 splits={ns}")
        assert_lse_close(LSE.cpu().numpy(), Lr, f"decode cfg0 lse splits={ns}")


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_decode_gqa_groups(G):
    O, LSE, Or, Lr = _decode_case(2, 2 * G, 2, 64 * 13, seed=40 + G)
    assert_close(O, Or, f"decode G={G}")
    assert_lse_close(LSE, Lr, f"decode G={G} lse")


def test_decode_all_dense_is_plain_attention():
    B, Hq, Hkv, L = 1, 8, 2, 64 * 9
    O, LSE, Or, Lr = _decode_case(B, Hq, Hkv, L, seed=50, sparse_frac_k=0.0, sparse_frac_v=0.0)
    assert_close(O, Or, "decode dense")
    # and against the library routine directly
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=50)
    f = lambda x: torch.from_numpy(wl.bf16_bits_to_f32(x).astype(np.float64))
    ref = torch.nn.functional.scaled_dot_product_attention(
        f(Q), f(K).repeat_interleave(4, 1), f(V).repeat_interleave(4, 1))[:, :, 0].numpy()
    assert_close(O, ref, "decode dense vs sdpa")


@pytest.mark.parametrize("sfk,sfv", [(0.0, 1.0), (1.0, 0.0), (0.5, 1.0), (0.0, 0.4)])
def test_decode_and_prefill_per_tensor_kinds(sfk, sfv):
    """Keys dense / values 2:4 (the paper's quality-preserving setting) and the other combinations
    that select per-tensor specialised kernels."""
    O, LSE, Or, Lr = _decode_case(1, 8, 2, 64 * 12, seed=65, sparse_frac_k=sfk, sparse_frac_v=sfv)
    assert_close(O, Or, f"decode S_K={sfk} S_V={sfv}")
    assert_lse_close(LSE, Lr, f"decode S_K={sfk} S_V={sfv} lse")
    O, LSE, Or, Lr = _prefill_case(1, 8, 2, 64 * 6, 64 * 6, seed=66, sparse_frac_k=sfk, sparse_frac_v=sfv)
    assert_close(O, Or, f"prefill S_K={sfk} S_V={sfv}")
    assert_lse_close(LSE, Lr, f"prefill S_K={sfk} S_V={sfv} lse")


def test_decode_mixed_and_skip():
    B, Hq, Hkv, L = 2, 8, 2, 64 * 21
    sk, sv = _mixed_states(B, Hkv, L // 64, seed=61)
    sk[1, 1, :] = 0     # one row with every tile skipped: O = 0, LSE = -inf
    sv[1, 1, :] = 0
    O, LSE, Or, Lr = _decode_case(B, Hq, Hkv, L, seed=60, state_k=sk, state_v=sv, n_splits=3)
    assert (O[1, 4:8] == 0).all() and np.isneginf(LSE[1, 4:8]).all()
    assert_close(O, Or, "decode mixed")
    assert_lse_close(LSE, Lr, "decode mixed lse")


@pytest.mark.parametrize("skip", [0.25, 0.75])
def test_decode_skip_policy_outlier_keys(skip):
    O, LSE, Or, Lr = _decode_case(1, 32, 8, 64 * 64, seed=70, k_outliers=True, skip_frac=skip)
    assert_close(O, Or, f"decode skip={skip}")
    assert_lse_close(LSE, Lr, f"decode skip={skip} lse")


# Rows long enough for the library to hand the kept tiles out by count (from 128 tiles per split with all-2:4
# tensors, from 256 otherwise): every wave gets the same number of tiles whatever the skip pattern.  The results
# must not depend on it.
@pytest.mark.parametrize("n_splits", [1, 2, 3, 7])
@pytest.mark.parametrize("pol", [dict(skip_frac=0.5), dict(skip_frac=0.75, sparse_frac_k=0.5, sparse_frac_v=0.25),
                                 dict(skip_frac=0.3, sparse_frac_k=0.0, sparse_frac_v=1.0)])
def test_decode_tiles_handed_out_by_count(pol, n_splits):
    O, LSE, Or, Lr = _decode_case(2, 8, 2, 64 * 512, seed=75, n_splits=n_splits, k_outliers=True, **pol)
    assert_close(O, Or, f"decode by count {pol} splits={n_splits}")
    assert_lse_close(LSE, Lr, f"decode by count {pol} splits={n_splits} lse")


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_decode_by_count_explicit_states_with_empty_and_nearly_empty_rows(dtype):
    B, Hq, Hkv, L = 2, 8, 2, 64 * 520
    T = L // 64
    sk, sv = _mixed_states(B, Hkv, T, seed=76, p_skip=0.6)
    sk[0, 1, :] = 0                       # a row with nothing kept
    sv[0, 1, :] = 0
    sk[1, 0, :] = 0                       # a row with fewer kept tiles (1) than splits (2): one split gets none
    sv[1, 0, :] = 0
    sk[1, 0, 77] = 2
    sv[1, 0, 77] = 1
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=77, dtype=dtype)
    if dtype == "bf16":                   # both V encodings in one row: a few values fp16 cannot hold
        V = V.copy()
        V[:, :, 64 * 5 + 3, 9] = 0x0080   # 2^-126
        V[:, :, 64 * 350 + 1, 100] = 0x4780   # 65536
    q = Q[:, :, 0, :].copy()
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, dtype=dtype, state_k=sk, state_v=sv)
    Or, Lr = orc.attention_decode(q, pk, pv)
    for ns in (1, 2):
        O, LSE = hb.decode_attn(sh, _dev(q, dtype), kv, n_splits=ns)
        torch.cuda.synchronize()
        O, LSE = _f32(O), LSE.cpu().numpy()
        assert (O[0, 4:8] == 0).all() and np.isneginf(LSE[0, 4:8]).all()
        assert_close(O, Or, f"decode by count mixed {dtype} splits={ns}")
        assert_lse_close(LSE, Lr, f"decode by count mixed {dtype} splits={ns} lse")


@pytest.mark.parametrize("n_splits", [1, 3])
def test_decode_by_count_row_longer_than_one_scan_step_and_one_list(n_splits):
    """4608 tiles in a row: three scan steps of 2048 tiles; with one split its 3456 kept tiles fill the
    workgroup's list of 2048 twice."""
    B, Hq, Hkv, L = 1, 2, 1, 64 * 4608
    O, LSE, Or, Lr = _decode_case(B, Hq, Hkv, L, seed=78, n_splits=n_splits, skip_frac=0.25)
    assert_close(O, Or, f"decode long row splits={n_splits}")
    assert_lse_close(LSE, Lr, f"decode long row splits={n_splits} lse")


def test_decode_by_count_with_a_dense_tail():
    """The dense tail's partial sits behind the cache splits whichever way the tiles are handed out."""
    B, Hq, Hkv, L = 1, 8, 2, 64 * 300
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L + 64, 128, 1, seed=79)
    q = Q[:, :, 0, :].copy()
    Kc, Vc, Kt, Vt = K[:, :, :L].copy(), V[:, :, :L].copy(), K[:, :, L:].copy(), V[:, :, L:].copy()
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, Kc, Vc, skip_frac=0.6)
    for ns in (1, 2):      # 300 and 150 tiles per split: by count
        O, LSE = hb.decode_attn(sh, _dev(q), kv, n_splits=ns, tail_k=_dev(Kt), tail_v=_dev(Vt), tail_len=23)
        torch.cuda.synchronize()
        Or, Lr = orc.attention_decode(q, pk, pv, tail_k=Kt, tail_v=Vt, tail_len=23)
        assert_close(_f32(O), Or, f"decode by count with tail, splits {ns}")
        assert_lse_close(LSE.cpu().numpy(), Lr, "decode by count with tail lse")


def test_decode_cfg1_full_size():
    """The benchmark workload at full size, in the launch configuration the benchmark times."""
    c, q, K, V = wl.make_config("cfg1_decode_llama8b_32k")
    sh = hb.make_shape(c["B"], c["Hq"], c["Hkv"], c["L"])
    Kd, Vd = _dev(K), _dev(V)
    kv = hb.compress_kv(sh, hb.make_policy(), Kd, Vd)
    O, LSE = hb.decode_attn(sh, _dev(q), kv)
    kvd = hb.compress_kv(sh, hb.make_policy(sparse_frac_k=0.0, sparse_frac_v=0.0), Kd, Vd)
    Od, LSEd = hb.decode_attn(sh, _dev(q), kvd)
    torch.cuda.synchronize()
    pk, pv, _ = orc.compress_kv(K, V)
    Or, Lr = orc.attention_decode(q, pk, pv)
    assert_close(_f32(O), Or, "decode cfg1 2:4")
    assert_lse_close(LSE.cpu().numpy(), Lr, "decode cfg1 lse")
    st = np.full((c["B"], c["Hkv"], c["L"] // 64), 1, dtype=np.int8)
    pk, pv, _ = orc.compress_kv(K, V, state_k=st, state_v=st)
    Or, Lr = orc.attention_decode(q, pk, pv)
    assert_close(_f32(Od), Or, "decode cfg1 dense")


# ------------------------------------------------------------------ prefill
def _prefill_case(B, Hq, Hkv, L, Lq, seed, causal=True, rows=None, **pol):
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, Lq, seed=seed)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, **pol)
    O, LSE = _prefill(sh, _dev(Q), kv, causal=causal)
    torch.cuda.synchronize()
    if rows is None:
        rows = [(b, h, i) for b in range(B) for h in range(Hq) for i in range(Lq)]
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=causal)
    idx = tuple(np.array(rows).T)
    return _f32(O)[idx], LSE.cpu().numpy()[idx], Or, Lr


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_prefill_causal_gqa_groups(G):
    O, LSE, Or, Lr = _prefill_case(1, 2 * G, 2, 64 * 5, 64 * 5, seed=80 + G)
    assert_close(O, Or, f"prefill G={G}")
    assert_lse_close(LSE, Lr, f"prefill G={G} lse")


def test_prefill_all_dense_and_noncausal():
    O, LSE, Or, Lr = _prefill_case(2, 4, 1, 64 * 4, 64 * 4, seed=90, sparse_frac_k=0.0, sparse_frac_v=0.0)
    assert_close(O, Or, "prefill dense causal")
    O, LSE, Or, Lr = _prefill_case(1, 4, 1, 64 * 4, 64 * 4, seed=91, causal=False)
    assert_close(O, Or, "prefill 2:4 non-causal")
    assert_lse_close(LSE, Lr, "prefill non-causal lse")


def test_prefill_mixed_skip_and_empty_rows():
    B, Hq, Hkv, L = 1, 8, 2, 64 * 9
    sk, sv = _mixed_states(B, Hkv, L // 64, seed=101, p_skip=0.3)
    sk[0, 0, 0] = sv[0, 0, 0] = 0      # first tile skipped: rows 0..63 of heads 0..3 see nothing
    sk[0, 0, 1] = sv[0, 0, 1] = 0
    sk[0, 1, 0] = 2
    sv[0, 1, 0] = 1
    O, LSE, Or, Lr = _prefill_case(B, Hq, Hkv, L, L, seed=100, state_k=sk, state_v=sv)
    assert_close(O, Or, "prefill mixed")
    assert_lse_close(LSE, Lr, "prefill mixed lse")
    assert np.isneginf(Lr).sum() >= 4 * 128


def test_prefill_chunk_lq_less_than_l():
    O, LSE, Or, Lr = _prefill_case(1, 8, 2, 64 * 8, 64 * 3, seed=110, skip_frac=0.25)
    assert_close(O, Or, "prefill Lq<L")
    assert_lse_close(LSE, Lr, "prefill Lq<L lse")


@pytest.mark.parametrize("q_start,Lq", [(0, 64 * 7), (64 * 5, 64 * 2), (64 * 3 + 17, 64 * 2), (64 * 12 - 64, 64)])
def test_prefill_queries_placed_inside_a_capacity_cache(q_start, Lq):
    """A cache allocated for 12 tiles that holds 7 so far (the rest SKIP): queries stand where the caller
    says (chunked prefill, growing caches), not at the end of the capacity.  Positions that are not a
    multiple of the tile, and queries beyond the filled part (they see everything filled), included."""
    B, Hq, Hkv, T_cap, T_now = 2, 8, 2, 12, 7
    L = 64 * T_cap
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, Lq, seed=250, k_outliers=True)
    sk, sv = _mixed_states(B, Hkv, T_cap, seed=251, p_skip=0.1)
    sk[:, :, T_now:], sv[:, :, T_now:] = 0, 0
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, state_k=sk, state_v=sv)
    O, LSE = _prefill(sh, _dev(Q), kv, q_start=q_start)
    torch.cuda.synchronize()
    rows = [(b, h, i) for b in range(B) for h in range(Hq) for i in range(Lq)]
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True, q_offset=q_start)
    idx = tuple(np.array(rows).T)
    assert_close(_f32(O)[idx], Or, f"prefill at {q_start}")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, f"prefill at {q_start} lse")
    if q_start == 0:
        for bad in (-1, L - Lq + 1):
            with pytest.raises(hb.HsError):
                hb.prefill_attn(sh, _dev(Q), kv, q_start=bad)


@pytest.mark.parametrize("slab", [None, 16, 32])                  # None: what the library picks for the room it gets
@pytest.mark.parametrize("n_ranges", [2, 5, 0])                   # 0: as many as the library picks
@pytest.mark.parametrize("B,G,T,Lq,q_start,causal,dtype,pol", [
    (1, 4, 40, 64, None, True, "bf16", dict()),                            # a short turn at the end of a context
    (2, 3, 33, 128, 64 * 20 + 17, True, "fp16", dict(sparse_frac_k=0.0)),  # off the tile grid, a group with idle waves
    (1, 1, 70, 64, 0, False, "bf16", dict(sparse_frac_k=0.5, sparse_frac_v=0.5)),
    (1, 8, 48, 192, None, True, "bf16", "states"),                         # ranges without a kept tile, queries that see nothing
    (1, 4, 40, 128, 64 * 30 + 5, True, "fp16", dict()),
    (1, 2, 36, 64, None, True, "bf16", dict(sparse_frac_k=0.0, sparse_frac_v=0.0)),
    (1, 2, 36, 64, None, True, "bf16", dict(sparse_frac_v=0.0)),
    (1, 2, 36, 64, 64 * 2 + 63, True, "fp16", dict(dense_first_tiles=1, dense_last_tiles=4)),              # more ranges than tiles in sight
])
def test_prefill_tiles_cut_into_ranges(slab, n_ranges, B, G, T, Lq, q_start, causal, dtype, pol):
    import ctypes as C
    Hkv, L = 2, 64 * T
    Q, K, V = wl.make_qkv(B, G * Hkv, Hkv, L, 128, Lq, seed=900 + T, dtype=dtype)
    if pol == "states":
        sk, sv = _mixed_states(B, Hkv, T, seed=901)
        sk[:, 0, :T - 3] = sv[:, 0, :T - 3] = 0
        sk[:, 1, 5:15] = sv[:, 1, 5:15] = 0
        sk[:, 0, T - 3] = sv[:, 0, T - 3] = 0
        V[:, :, ::67, 5] = 0x0001                     # bf16 values that fp16 does not hold: both encodings
        pol = dict(state_k=sk, state_v=sv)
    sh, kv, pk, pv, _ = compress_both(B, G * Hkv, Hkv, L, K, V, dtype=dtype, **pol)
    Qd, at = _dev(Q, dtype), L - Lq if q_start is None else q_start
    need = hb.prefill_workspace_bytes(sh, Lq, at, kv, causal)
    one = B * G * Hkv * Lq * 129 * 4
    n = n_ranges or max(need // one, 1)
    if q_start != 64 * 2 + 63:
        assert need >= 2 * one                        # the library does cut these shapes
    elif slab is not None:
        n = n_ranges or 8
    ws = torch.full((n * one + 64,), 255, dtype=torch.uint8, device="cuda")
    O, LSE = torch.full_like(Qd, float("nan")), torch.full(Qd.shape[:3], float("nan"), device="cuda")
    kvs = kv.struct()
    args = (C.byref(sh), Lq, at, 0.0, int(causal), hb._ptr(Qd), C.byref(kvs), hb._ptr(O), hb._ptr(LSE), hb._ptr(ws), n * one)
    if slab is None:
        assert hb.prefill_plan(sh, Lq, at, kv, causal, n * one)[1] <= n
        hb._check(hb.lib().hs_prefill_attn_ws(*args, hb._stream()))
    else:
        hb._check(hb.lib().hs_prefill_attn_planned(*args, slab, n, hb._stream()))
    torch.cuda.synchronize()
    assert (ws[n * one:] == 255).all()                # nothing past the bytes it was given
    rows = [(b, h, i) for b in range(B) for h in range(G * Hkv) for i in range(0, Lq, 3)]
    idx = tuple(np.array(rows).T)
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=causal, **({} if q_start is None else {"q_offset": q_start}))
    assert_close(_f32(O)[idx], Or, f"prefill in {n} ranges")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, f"prefill in {n} ranges lse")
    if n_ranges == 0 and slab is None:                # the binding's own call takes the same way
        O2, LSE2 = hb.prefill_attn(sh, Qd, kv, causal=causal, q_start=q_start)
        assert torch.equal(O2.view(torch.int16), O.view(torch.int16)) and torch.equal(LSE2, LSE)


@pytest.mark.parametrize("B,T,Lq,q_start,causal,G", [(1, 1, 64, None, True, 4), (1, 2, 128, None, True, 3), (1, 7, 64, 64 * 3 + 17, True, 1),
                                                      (1, 66, 128, None, True, 2), (1, 67, 64, 5, False, 5), (3, 8, 192, None, True, 2), (2, 5, 320, None, True, 7)])
@pytest.mark.parametrize("dtype,pol", [("bf16", dict()), ("fp16", dict()), ("bf16", "states"), ("fp16", "states"), ("fp16", dict(sparse_frac_k=0.0)),
                                       ("bf16", dict(sparse_frac_v=0.0)), ("bf16", dict(sparse_frac_k=0.0, sparse_frac_v=0.0)),
                                       ("bf16", dict(sparse_frac_k=0.5)), ("bf16", dict(sparse_frac_v=0.5, skip_frac=0.3))])
def test_prefill_two_teams_of_waves(B, T, Lq, q_start, causal, G, dtype, pol):
    """Two teams that take a workgroup's tiles in turn: no tile, one, an odd number, more than a window of the maps; every kind
    and both encodings of V; groups with idle waves; queries that see nothing; batches."""
    Hkv, L = 2, 64 * T
    Q, K, V = wl.make_qkv(B, G * Hkv, Hkv, L, 128, Lq, seed=1300 + T, dtype=dtype)
    V[:, 1, ::67, 5] = 0x0001                         # in bf16: values that fp16 does not hold
    if pol == "states":
        sk, sv = _mixed_states(B, Hkv, T, seed=1301)
        sk[:, 0, :T // 2] = sv[:, 0, :T // 2] = 0
        pol = dict(state_k=sk, state_v=sv)
    sh, kv, pk, pv, _ = compress_both(B, G * Hkv, Hkv, L, K, V, dtype=dtype, **pol)
    O, LSE = hb.prefill_attn_planned(sh, _dev(Q, dtype), kv, 16 | hb.TWO_TEAMS, 1, causal=causal, q_start=q_start)
    rows = [(b, h, i) for b in range(B) for h in range(G * Hkv) for i in range(0, Lq, 3)]
    idx = tuple(np.array(rows).T)
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=causal, **({} if q_start is None else {"q_offset": q_start}))
    assert_close(_f32(O)[idx], Or, "prefill by two teams")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "prefill by two teams lse")
    for slab, n in ((32 | hb.TWO_TEAMS, 1), (16 | hb.TWO_TEAMS, 2)):
        with pytest.raises(hb.HsError):
            hb.prefill_attn_planned(sh, _dev(Q, dtype), kv, slab, n)


@pytest.mark.parametrize("B,Hkv,L,Lq,plan", [(1, 8, 2048, 512, (16 | hb.TWO_TEAMS, 1)), (1, 8, 2048, 576, (16, 1)), (2, 2, 1024, 256, (16 | hb.TWO_TEAMS, 1)),
                                             (1, 8, 256, 128, (16, 1)), (1, 1, 4096, 4096, (16, 3)), (1, 8, 8192, 64, (16, 8))])
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_prefill_by_the_plan_that_is_told_is_the_call(B, Hkv, L, Lq, plan, dtype):
    """prefill_attn and the plan of prefill_plan_teams handed to prefill_attn_planned: the same bits."""
    sh = hb.make_shape(B, 4 * Hkv, Hkv, L, dtype=hb.FP16 if dtype == "fp16" else hb.BF16)
    g = torch.Generator(device="cuda").manual_seed(1320)
    K, V, Q = (torch.randn((B, h, n, 128), device="cuda", generator=g).to(hb.torch_dtype(sh)) for h, n in ((Hkv, L), (Hkv, L), (4 * Hkv, Lq)))
    kv = hb.compress_kv(sh, hb.make_policy(), K, V)
    slab, ranges, need = hb.prefill_plan_teams(sh, Lq, L - Lq, kv)
    assert (slab, ranges) == plan
    O, LSE = hb.prefill_attn(sh, Q, kv)
    O2, LSE2 = hb.prefill_attn_planned(sh, Q, kv, slab, ranges)
    assert torch.equal(O.view(torch.int16), O2.view(torch.int16)) and torch.equal(LSE, LSE2)


@pytest.mark.parametrize("dtype,pol", [("bf16", dict()), ("fp16", dict(sparse_frac_k=0.0)), ("bf16", dict(dense_first_tiles=1, dense_last_tiles=4)),
                                       ("fp16", dict(sparse_frac_k=0.5))])
def test_prefill_nan_scores_come_out_of_two_teams(dtype, pol):
    """A query that sees a NaN score, whichever team meets it, has O and LSE NaN; the others see nothing of it."""
    T, Lq = 9, 128
    Q, K, V, tok = _nan_case(T, Lq, dtype, 1310)
    sh = hb.make_shape(1, 4, 2, 64 * T, dtype=Q.dtype)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K.cuda(), V.cuda())
    Ku, Vu = (x.cpu() for x in hb.unpack_kv(sh, kv))
    Or, Lr = _nan_reference(Q[0], Ku[0], Vu[0], torch.arange(64 * T)[None, :] <= 64 * T - Lq + torch.arange(Lq)[:, None])
    O, LSE = hb.prefill_attn_planned(sh, Q.cuda(), kv, 16 | hb.TWO_TEAMS, 1)
    _check_nan_rows(O.cpu()[0], LSE.cpu()[0], Or, Lr, "two teams, NaN scores")


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("pol", [dict(), dict(sparse_frac_k=0.0), dict(sparse_frac_v=0.0), dict(sparse_frac_k=0.0, sparse_frac_v=0.0),
                                 dict(sparse_frac_k=0.5, sparse_frac_v=0.5), dict(sparse_frac_k=0.5), dict(dense_first_tiles=1, dense_last_tiles=1)])
def test_prefill_slabs_of_16_and_of_32_queries(pol, dtype):
    """The same prompts as one batch, whose workgroups fill the GPU twice with slabs of 32 queries, and one by one, too few for
    that, with slabs of 16: both against the oracle, every kind of tensor."""
    B, Hq, Hkv, L = 16, 32, 8, 256
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=1201, dtype=dtype)
    V[:, :, ::61, 3] = 0x0001                         # in bf16: values that fp16 does not hold, in every tile
    V[1::2] = wl.make_qkv(B // 2, Hq, Hkv, L, 128, L, seed=1202, dtype=dtype)[2]
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, dtype=dtype, **pol)
    wide, wide_l = hb.prefill_attn(sh, _dev(Q, dtype), kv)
    rows = wl.sample_rows(B, Hq, L, 600, seed=1203, extra=[(0, 0, 0), (1, 31, L - 1), (1, 5, 15), (0, 5, 16), (1, 6, 31), (0, 7, 63)])
    idx = tuple(np.array(rows).T)
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    assert_close(_f32(wide)[idx], Or, "slabs of 32")
    assert_lse_close(wide_l.cpu().numpy()[idx], Lr, "slabs of 32 lse")
    one, narrow, narrow_l = hb.make_shape(1, Hq, Hkv, L, dtype=sh.dtype), [], []
    for b in range(2):
        kv1 = hb.compress_kv(one, hb.make_policy(**pol), _dev(K[b:b + 1], dtype), _dev(V[b:b + 1], dtype))
        O, LSE = hb.prefill_attn(one, _dev(Q[b:b + 1], dtype), kv1)
        narrow.append(O)
        narrow_l.append(LSE)
    pick = np.array([r[0] < 2 for r in rows])
    idx = tuple(i[pick] for i in idx)
    assert_close(_f32(torch.cat(narrow))[idx], Or[pick], "slabs of 16")
    assert_lse_close(torch.cat(narrow_l).cpu().numpy()[idx], Lr[pick], "slabs of 16 lse")


@pytest.mark.parametrize("B,Hq,Hkv,L,Lq,q_start,causal", [
    (1, 5, 5, 192, 192, None, True),                  # groups of one head: a workgroup's waves at different positions
    (1, 21, 3, 320, 320, None, True),                 # 7 heads: slabs that do not divide among the waves
    (2, 6, 2, 640, 64, 64 * 4 + 33, True),            # off the tile grid
    (1, 8, 1, 1024, 64, None, False),                 # not causal, in ranges
    (1, 64, 8, 16384, 128, None, True),               # long enough that ranges of the wide slab are the better ones
])
def test_prefill_slab_choice_over_shapes(B, Hq, Hkv, L, Lq, q_start, causal):
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, Lq, seed=1210 + Hq, k_outliers=True)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V)
    O, LSE = _prefill(sh, _dev(Q), kv, causal=causal, q_start=q_start)
    rows = wl.sample_rows(B, Hq, Lq, 200, seed=1211, extra=[(0, 0, 0), (B - 1, Hq - 1, Lq - 1), (0, Hq - 1, 16), (0, 0, 15)])
    idx = tuple(np.array(rows).T)
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=causal, **({} if q_start is None else {"q_offset": q_start}))
    assert_close(_f32(O)[idx], Or, "slab choice")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "slab choice lse")


@pytest.mark.parametrize("q_start", [None, 64 * 20 + 17])
def test_prefill_entries_without_scratch_run_in_one_range(q_start, monkeypatch):
    """A shape the library would cut into ranges, through the entries that get no scratch, too little of it or none to
    be had: the one-range result, the same bits from each, and no write to a workspace that comes without a size."""
    import ctypes as C
    G, T, Lq, Hkv = 4, 40, 64, 2
    L = 64 * T
    Q, K, V = wl.make_qkv(1, G * Hkv, Hkv, L, 128, Lq, seed=931)
    sh, kv, pk, pv, _ = compress_both(1, G * Hkv, Hkv, L, K, V)
    Qd, at, kvs = _dev(Q), L - Lq if q_start is None else q_start, kv.struct()
    one = G * Hkv * Lq * 129 * 4
    assert hb.prefill_workspace_bytes(sh, Lq, at, kv) >= 2 * one
    ws = torch.full((8 * one,), 255, dtype=torch.uint8, device="cuda")
    lib, sp, q, w, st = hb.lib(), C.byref(sh), hb._ptr(Qd), hb._ptr(ws), hb._stream()
    calls = {"at": lambda o, l: lib.hs_prefill_attn_at(sp, Lq, at, 0.0, 1, q, C.byref(kvs), o, l, w, st),
             "no workspace": lambda o, l: lib.hs_prefill_attn_ws(sp, Lq, at, 0.0, 1, q, C.byref(kvs), o, l, None, 8 * one, st),
             "no bytes": lambda o, l: lib.hs_prefill_attn_ws(sp, Lq, at, 0.0, 1, q, C.byref(kvs), o, l, w, 0, st),
             "one range's bytes": lambda o, l: lib.hs_prefill_attn_ws(sp, Lq, at, 0.0, 1, q, C.byref(kvs), o, l, w, 2 * one - 1, st)}
    if q_start is None:
        calls["end"] = lambda o, l: lib.hs_prefill_attn(sp, Lq, 0.0, 1, q, C.byref(kvs), o, l, w, st)
    got = {}
    for name, call in calls.items():
        O, LSE = torch.full_like(Qd, float("nan")), torch.full(Qd.shape[:3], float("nan"), device="cuda")
        hb._check(call(hb._ptr(O), hb._ptr(LSE)))
        got[name] = O, LSE
    def full(nbytes, device):
        raise torch.OutOfMemoryError("no scratch to be had")
    monkeypatch.setattr(hb, "_workspace", full)
    got["out of memory"] = hb.prefill_attn(sh, Qd, kv, q_start=q_start)
    torch.cuda.synchronize()
    assert (ws == 255).all()
    rows = [(0, h, i) for h in range(G * Hkv) for i in range(0, Lq, 3)]
    idx = tuple(np.array(rows).T)
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True, q_offset=at)
    O0, L0 = got["at"]
    assert_close(_f32(O0)[idx], Or, "prefill without scratch")
    assert_lse_close(L0.cpu().numpy()[idx], Lr, "prefill without scratch lse")
    for name, (O, LSE) in got.items():
        assert torch.equal(O.view(torch.int16), O0.view(torch.int16)) and torch.equal(LSE, L0), name


def test_calls_go_to_the_current_stream(monkeypatch):
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            handle = hb._stream()
            with monkeypatch.context() as m:
                m.setattr(hb, "_raw_stream", None)
                assert handle == hb._stream() == stream.cuda_stream


def test_decode_equals_last_prefill_row():
    B, Hq, Hkv, L = 1, 8, 2, 64 * 6
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=120)
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv = hb.compress_kv(sh, hb.make_policy(), _dev(K), _dev(V))
    O, _ = hb.prefill_attn(sh, _dev(Q), kv)
    Od, _ = hb.decode_attn(sh, _dev(Q[:, :, -1, :].copy()), kv)
    torch.cuda.synchronize()
    assert_close(_f32(Od), _f32(O)[:, :, -1, :], "decode vs last prefill row")


def test_prefill_cfg2_full_size_sampled_rows():
    c, Q, K, V = wl.make_config("cfg2_prefill_llama8b_16k")
    rows = wl.sample_rows(c["B"], c["Hq"], c["L"], 256, seed=c["seed"] + 4,
                          extra=[(0, 0, 0), (0, 31, c["L"] - 1), (0, 5, 63), (0, 5, 64)])
    sh = hb.make_shape(c["B"], c["Hq"], c["Hkv"], c["L"])
    kv = hb.compress_kv(sh, hb.make_policy(), _dev(K), _dev(V))
    O, LSE = hb.prefill_attn(sh, _dev(Q), kv)
    torch.cuda.synchronize()
    pk, pv, _ = orc.compress_kv(K, V)
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    assert_close(_f32(O)[idx], Or, "prefill cfg2 sampled")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "prefill cfg2 lse")


@pytest.mark.parametrize("pol", [dict(), dict(sparse_frac_k=0.0, sparse_frac_v=1.0)])
def test_prefill_on_the_benchmark_workload_full_size_sampled_rows(pol):
    """Causal prefill on the inputs the benchmark's step times (L = 32768, keys with outlier channels, which
    drive the lazily renewed softmax reference through its redo path), all tiles 2:4 and keys dense /
    values 2:4: 160 seeded rows plus the first and last row and the rows around the first tile edge."""
    c = wl.CONFIGS["cfg1_decode_llama8b_32k"]
    B, Hq, Hkv, L = c["B"], c["Hq"], c["Hkv"], c["L"]
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, c["D"], L, c["seed"], c["k_outliers"])
    rows = wl.sample_rows(B, Hq, L, 160, seed=c["seed"] + 4,
                          extra=[(0, 0, 0), (0, Hq - 1, L - 1), (0, 7, 63), (0, 7, 64), (0, 13, L - 65)])
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), _dev(K), _dev(V))
    O, LSE = hb.prefill_attn(sh, _dev(Q), kv)
    torch.cuda.synchronize()
    pk, pv, _ = orc.compress_kv(K, V, **pol)
    assert_maps_equal(kv, pk, pv)
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    assert_close(_f32(O)[idx], Or, f"prefill benchmark workload {sorted(pol)}")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "prefill benchmark workload lse")


def test_decode_cfg3_shape_one_batch_row_skip75():
    """Hierarchical decode sweep workload (L = 131072, 32/8 heads) at its full context for one
    batch row, 75 % of the tiles skipped + 2:4 in the rest, default launch configuration."""
    c, q, K, V = wl.make_config("cfg3_decode_b8_128k", B=1)
    sh, kv, pk, pv, info = compress_both(c["B"], c["Hq"], c["Hkv"], c["L"], K, V, skip_frac=0.75)
    assert_maps_equal(kv, pk, pv)
    assert int((pk.map == 0).sum()) == 8 * 1536
    O, LSE = hb.decode_attn(sh, _dev(q), kv)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, pk, pv)
    assert_close(_f32(O), Or, "decode cfg3 B=1 skip 0.75")
    assert_lse_close(LSE.cpu().numpy(), Lr, "decode cfg3 lse")


@pytest.mark.parametrize("pol", [dict(skip_frac=0.25), dict(skip_frac=0.5), dict(skip_frac=0.75),
                                 dict(sparse_frac_k=0.0, sparse_frac_v=1.0)])
def test_decode_cfg3_full_batch_sampled_rows(pol):
    """The hierarchical decode workload at its full size (B = 8, L = 131072: 4.3 GB of K and V, pools past
    2^31 bytes), default launch configuration.  Inputs are drawn on the device (seeded); the oracle
    compresses and attends three sampled (batch, kv head) rows, each of which is ranked on its own."""
    B, Hq, Hkv, L = 8, 32, 8, 131072
    g = torch.Generator(device="cuda")
    g.manual_seed(300)
    K = torch.randn((B, Hkv, L, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    V = torch.randn((B, Hkv, L, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    q = torch.randn((B, Hq, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K, V)
    O, LSE = hb.decode_attn(sh, q, kv)
    torch.cuda.synchronize()
    G = Hq // Hkv
    for b, h in ((0, 0), (3, 5), (7, 7)):
        print(f"[cfg3 full batch {sorted(pol)}] row b={b} hkv={h}", flush=True)
        Kb, Vb = hb.bf16_tensor_to_bits(K[b:b + 1, h:h + 1]), hb.bf16_tensor_to_bits(V[b:b + 1, h:h + 1])
        pk, pv, _ = orc.compress_kv(Kb, Vb, Bt=64, **pol)
        assert_maps_equal(kv, pk, pv, sel=(b, h), osel=(0, 0))
        for p, dense, nnz, meta, cd, cs in ((pk, kv.k_dense, kv.k_nnz, kv.k_meta, kv.counts[1], kv.counts[2]),
                                            (pv, kv.v_dense, kv.v_nnz, kv.v_meta, kv.counts[3], kv.counts[4])):
            ph = hl.physical_pools(p)
            nd, ns = int(ph["n_dense"][0, 0]), int(ph["n_sparse"][0, 0])
            for slot in {0, nd // 2, nd - 1} - {-1}:           # first, middle and last used slot
                if nd:
                    assert (dense.view(B, Hkv, cd, 16384)[b, h, slot].cpu().numpy() == ph["dense"][0, 0, slot]).all()
            for slot in {0, ns // 2, ns - 1} - {-1}:
                if ns:
                    assert (nnz.view(B, Hkv, cs, 8192)[b, h, slot].cpu().numpy() == ph["nnz"][0, 0, slot]).all()
                    assert (meta.view(B, Hkv, cs, 1024)[b, h, slot].cpu().numpy() == ph["meta"][0, 0, slot]).all()
        qb = hb.bf16_tensor_to_bits(q[b:b + 1, G * h:G * (h + 1)])
        Or, Lr = orc.attention_decode(qb, pk, pv)
        assert_close(_f32(O[b:b + 1, G * h:G * (h + 1)]), Or, f"decode cfg3 full batch b{b} hkv{h}")
        assert_lse_close(LSE[b:b + 1, G * h:G * (h + 1)].cpu().numpy(), Lr, "decode cfg3 full batch lse")


def _check_sampled_heads(sh, kv, K, V, Q, O, LSE, q_dec, O_dec, LSE_dec, pol, heads, n_rows, seed, dtype="bf16", q_start=None):
    """Oracle check of device-generated full-size inputs on sampled (batch, kv head) rows: maps and a few pool
    slots bit for bit, prefill on n_rows sampled queries of one query head of the group, decode on the group."""
    B, Hq, Hkv, L = sh.B, sh.Hq, sh.Hkv, sh.L
    G = Hq // Hkv
    rng = np.random.default_rng(seed)
    for b, h in heads:
        print(f"[sampled heads] b={b} hkv={h} {sorted(pol)}", flush=True)
        Kb, Vb = hb.bf16_tensor_to_bits(K[b:b + 1, h:h + 1]), hb.bf16_tensor_to_bits(V[b:b + 1, h:h + 1])
        pk, pv, _ = orc.compress_kv(Kb, Vb, Bt=64, dtype=dtype, **pol)
        assert_maps_equal(kv, pk, pv, sel=(b, h), osel=(0, 0))
        if Q is not None:
            Lq = Q.shape[2]
            hq = G * h + int(rng.integers(G))
            qi = sorted(set([0, Lq - 1] + [int(x) for x in rng.integers(0, Lq, size=n_rows)]))
            Qb = hb.bf16_tensor_to_bits(Q[b:b + 1, hq:hq + 1])
            Or, Lr = orc.attention_rows(Qb, pk, pv, [(0, 0, i) for i in qi], causal=True, q_offset=q_start)
            assert_close(_f32(O[b, hq])[qi], Or, f"prefill sampled b{b} hq{hq}")
            assert_lse_close(LSE[b, hq].cpu().numpy()[qi], Lr, f"prefill sampled lse b{b} hq{hq}")
        if q_dec is not None:
            qb = hb.bf16_tensor_to_bits(q_dec[b:b + 1, G * h:G * (h + 1)])
            Or, Lr = orc.attention_decode(qb, pk, pv)
            assert_close(_f32(O_dec[b:b + 1, G * h:G * (h + 1)]), Or, f"decode sampled b{b} hkv{h}")
            assert_lse_close(LSE_dec[b:b + 1, G * h:G * (h + 1)].cpu().numpy(), Lr, f"decode sampled lse b{b} hkv{h}")


@pytest.mark.parametrize("pol", [dict(), dict(sparse_frac_k=0.0, sparse_frac_v=1.0)])
def test_paper_kernel_shape_b8_32k_sampled_heads(pol):
    """The shape of the paper's own kernel benchmarks (Sec. V-B: batch 8, 32K tokens, 32 / 8 heads) at full size,
    as the benchmark leg runs it: prefill and decode, all tiles 2:4 and keys dense / values 2:4, against the
    oracle on two sampled (batch, kv head) rows."""
    B, Hq, Hkv, L = 8, 32, 8, 32768
    g = torch.Generator(device="cuda")
    g.manual_seed(500)
    K = torch.randn((B, Hkv, L, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    V = torch.randn((B, Hkv, L, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    Q = torch.randn((B, Hq, L, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K, V)
    O, LSE = hb.prefill_attn(sh, Q, kv)
    q = Q[:, :, -1, :].contiguous()
    Od, LSEd = hb.decode_attn(sh, q, kv)
    torch.cuda.synchronize()
    _check_sampled_heads(sh, kv, K, V, Q, O, LSE, q, Od, LSEd, pol, [(0, 0), (6, 5)], 24, seed=501)


def test_fp16_benchmark_shape_sampled_heads():
    """fp16 (the paper's element type) at the benchmark workload's shape (L = 32768), as the fp16 leg runs it."""
    B, Hq, Hkv, L = 1, 32, 8, 32768
    g = torch.Generator(device="cuda")
    g.manual_seed(510)
    K = torch.randn((B, Hkv, L, 128), device="cuda", dtype=torch.float16, generator=g)
    V = torch.randn((B, Hkv, L, 128), device="cuda", dtype=torch.float16, generator=g)
    Q = torch.randn((B, Hq, L, 128), device="cuda", dtype=torch.float16, generator=g)
    sh = hb.make_shape(B, Hq, Hkv, L, dtype=hb.FP16)
    for pol in (dict(), dict(sparse_frac_k=0.0, sparse_frac_v=1.0)):
        kv = hb.compress_kv(sh, hb.make_policy(**pol), K, V)
        O, LSE = hb.prefill_attn(sh, Q, kv)
        q = Q[:, :, -1, :].contiguous()
        Od, LSEd = hb.decode_attn(sh, q, kv)
        torch.cuda.synchronize()
        _check_sampled_heads(sh, kv, K, V, Q, O, LSE, q, Od, LSEd, pol, [(0, 3)], 32, seed=511, dtype="fp16")


def test_chunked_prefill_128k_in_32k_chunks_sampled_head():
    """Chunked prefill as the benchmark leg runs it (a cache allocated for 128K tokens, 32K-token chunks, per
    chunk one append and one causal attention call at the chunk's position): the last chunk's outputs and the
    final cache against the oracle on one sampled kv head."""
    Hq, Hkv, Lc, chunk = 32, 8, 131072, 32768
    Tc, nct = Lc // 64, chunk // 64
    g = torch.Generator(device="cuda")
    g.manual_seed(520)
    K = torch.randn((1, Hkv, Lc, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    V = torch.randn((1, Hkv, Lc, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    Q = torch.randn((1, Hq, chunk, 128), device="cuda", dtype=torch.bfloat16, generator=g)
    sh = hb.make_shape(1, Hq, Hkv, Lc)
    kv = hb.PackedKV(sh, [0, Tc, 0, 0, Tc])                  # keys dense, values 2:4
    kv.uniform = 0
    kv.k_map.zero_()
    kv.v_map.zero_()
    ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
    for c in range(Lc // chunk):
        hb.append_tile(sh, kv, nct * c, K[:, :, chunk * c:chunk * (c + 1)], V[:, :, chunk * c:chunk * (c + 1)],
                       state_k=hb.DENSE, state_v=hb.SPARSE24, overflow=ovf)
        O, LSE = hb.prefill_attn(sh, Q, kv, q_start=chunk * c)
    torch.cuda.synchronize()
    assert int(ovf.item()) == 0
    pol = dict(sparse_frac_k=0.0, sparse_frac_v=1.0)          # what the appended states amount to
    _check_sampled_heads(sh, kv, K, V, Q, O, LSE, None, None, None, pol, [(0, 6)], 12, seed=521, q_start=Lc - chunk)


def test_selection_on_a_row_longer_than_the_register_cache():
    """Tile selection with more than 8 tiles per thread (rows over 2048 tiles take the path that re-reads
    the scores instead of holding them in registers): maps against the oracle, with planted equal tiles
    so that ties on the cut are broken by tile index."""
    B, Hq, Hkv, T = 1, 1, 1, 2304
    L = 64 * T
    rng = np.random.default_rng(240)
    K = wl.f32_to_bf16_bits(rng.standard_normal((B, Hkv, L, 128)).astype(np.float32))
    V = wl.f32_to_bf16_bits(rng.standard_normal((B, Hkv, L, 128)).astype(np.float32))
    for t in (7, 900, 2200):                                 # the three quietest tiles are identical
        K[0, 0, 64 * t:64 * t + 64] = K[0, 0, 64 * 7:64 * 7 + 64] & 0x8000 | 0x3000
        V[0, 0, 64 * t:64 * t + 64] = V[0, 0, 64 * 7:64 * 7 + 64] & 0x8000 | 0x3000
    pol = dict(skip_frac=2 / (T - 4) + 1e-9, sparse_frac_k=0.5, sparse_frac_v=0.7, dense_first_tiles=1, dense_last_tiles=3)
    sh, kv, pk, pv, info = compress_both(B, Hq, Hkv, L, K, V, **pol)
    assert int((pk.map == 0).sum()) == 2 and pk.map[0, 0, 7] == 0 and pk.map[0, 0, 900] == 0 and pk.map[0, 0, 2200] != 0
    assert_maps_equal(kv, pk, pv)
    Ku, Vu = hb.unpack_kv(sh, kv)
    torch.cuda.synchronize()
    assert (hb.bf16_tensor_to_bits(Ku) == orc.unpack_tensor(pk)).all()
    assert (hb.bf16_tensor_to_bits(Vu) == orc.unpack_tensor(pv)).all()


def test_prefill_cfg4_full_size_skip75_sampled_rows():
    """Long causal prefill at the highest hierarchical sparsity (L = 65536, 75 % of the tiles
    skipped, 2:4 in the rest): seeded sampled rows plus rows that see no token at all."""
    c, Q, K, V = wl.make_config("cfg4_prefill_64k")
    sh, kv, pk, pv, info = compress_both(c["B"], c["Hq"], c["Hkv"], c["L"], K, V, skip_frac=0.75)
    assert_maps_equal(kv, pk, pv)
    # rows whose own and all earlier tiles are skipped (kv head 0 ... 7): O = 0, LSE = -inf
    extra = []
    for hkv in range(c["Hkv"]):
        first_kept = int(np.nonzero(pk.map[0, hkv] != 0)[0][0])
        if first_kept > 0:
            extra += [(0, 4 * hkv, 0), (0, 4 * hkv + 3, 64 * first_kept - 1)]
        extra += [(0, 4 * hkv + 1, 64 * first_kept), (0, 4 * hkv + 2, c["L"] - 1)]
    rows = wl.sample_rows(c["B"], c["Hq"], c["L"], 160, seed=c["seed"] + 4, extra=extra)
    O, LSE = hb.prefill_attn(sh, _dev(Q), kv)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    got, lse = _f32(O)[idx], LSE.cpu().numpy()[idx]
    empty = np.isneginf(Lr)
    assert empty.sum() >= 1
    assert (got[empty] == 0).all()
    assert_close(got, Or, "prefill cfg4 skip 0.75 sampled")
    assert_lse_close(lse, Lr, "prefill cfg4 lse")


def test_decode_with_dense_tail():
    """Cache of whole tiles plus 0..64 recent tokens that are not compressed yet."""
    B, Hq, Hkv, L = 2, 8, 2, 64 * 7
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L + 64, 128, 1, seed=160)
    q = Q[:, :, 0, :].copy()
    Kc, Vc, Kt, Vt = K[:, :, :L].copy(), V[:, :, :L].copy(), K[:, :, L:].copy(), V[:, :, L:].copy()
    sk, sv = _mixed_states(B, Hkv, L // 64, seed=161, p_skip=0.3)
    for pol in (dict(), dict(state_k=sk, state_v=sv)):
        sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, Kc, Vc, **pol)
        for tail_len in (0, 1, 17, 64):
            for ns in (0, 3):
                O, LSE = hb.decode_attn(sh, _dev(q), kv, n_splits=ns, tail_k=_dev(Kt), tail_v=_dev(Vt), tail_len=tail_len)
                torch.cuda.synchronize()
                Or, Lr = orc.attention_decode(q, pk, pv, tail_k=Kt, tail_v=Vt, tail_len=tail_len)
                assert_close(_f32(O), Or, f"decode tail {tail_len} splits {ns} {sorted(pol)}")
                assert_lse_close(LSE.cpu().numpy(), Lr, f"decode tail {tail_len} lse")
    # every cached tile skipped: the tail alone answers
    z = np.zeros((B, Hkv, L // 64), dtype=np.int8)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, Kc, Vc, state_k=z, state_v=z)
    O, LSE = hb.decode_attn(sh, _dev(q), kv, tail_k=_dev(Kt), tail_v=_dev(Vt), tail_len=5)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, pk, pv, tail_k=Kt, tail_v=Vt, tail_len=5)
    assert_close(_f32(O), Or, "decode tail only")
    assert_lse_close(LSE.cpu().numpy(), Lr, "decode tail only lse")
    import ctypes as C
    kvs = kv.struct()
    qd = _dev(q)
    assert hb.lib().hs_decode_attn_tail(C.byref(sh), 0.0, 0, hb._ptr(qd), C.byref(kvs), None, None, 65, hb._ptr(qd), None,
                                        hb._ptr(qd), None) == -1
    assert hb.lib().hs_decode_attn_tail(C.byref(sh), 0.0, 0, hb._ptr(qd), C.byref(kvs), None, None, 3, hb._ptr(qd), None,
                                        hb._ptr(qd), None) == -1


@pytest.mark.parametrize("B,Hkv,G,T,n_splits,dtype", [(3, 2, 1, 1, 1, "bf16"), (5, 1, 3, 4, 2, "fp16"), (2, 3, 8, 6, 4, "bf16"),
                                                       (7, 2, 5, 3, 1, "fp16")])
def test_decode_tail_workgroups_of_every_row(B, Hkv, G, T, n_splits, dtype):
    """Tail lengths of every kind side by side (none, one token, both sides of a 16-token block, all 64) and
    numbers of rows that do and do not fill the last plane of tail workgroups."""
    lens = [0, 1, 15, 16, 17, 63, 64][:B]
    L = 64 * T
    Q, K, V = wl.make_qkv(B, G * Hkv, Hkv, L + 64, 128, 1, seed=950 + B, dtype=dtype)
    q, Kc, Vc, Kt, Vt = Q[:, :, 0].copy(), K[:, :, :L].copy(), V[:, :, :L].copy(), K[:, :, L:].copy(), V[:, :, L:].copy()
    sh, kv, pk, pv, _ = compress_both(B, G * Hkv, Hkv, L, Kc, Vc, dtype=dtype)
    tk, tv = _dev(Kt, dtype), _dev(Vt, dtype)
    for b, n in enumerate(lens):                      # tokens past a row's tail must not be looked at
        tk[b, :, n:], tv[b, :, n:] = float("nan"), float("nan")
    rows = torch.tensor(lens, dtype=torch.int32, device="cuda")
    O, LSE = hb.decode_attn(sh, _dev(q, dtype), kv, n_splits=n_splits, tail_k=tk, tail_v=tv, tail_len=rows)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        Or, Lr = orc.attention_decode(q, pk, pv, tail_k=Kt, tail_v=Vt, tail_len=n)
        assert_close(_f32(O)[b], Or[b], f"decode tail of {n} in row {b}")
        assert_lse_close(LSE.cpu().numpy()[b], Lr[b], f"decode tail of {n} in row {b} lse")


@pytest.mark.parametrize("B,Hkv,G,T,dtype,pol", [
    (7, 1, 1, 1, "bf16", dict()), (7, 2, 8, 6, "fp16", dict()), (7, 1, 5, 7, "bf16", dict()),            # one workgroup a row | splits
    (7, 1, 4, 4, "fp16", dict(sparse_frac_k=0.0, sparse_frac_v=0.0)), (7, 1, 3, 5, "bf16", dict(sparse_frac_k=0.0)),
    (7, 3, 7, 3, "bf16", dict(dense_first_tiles=1, dense_last_tiles=4)), (7, 19, 2, 16, "bf16", dict())])
def test_decode_tail_in_the_rows_own_workgroup(B, Hkv, G, T, dtype, pol):
    """The library's choice of route on both sides of its edges, with tails of every kind; every workgroup's 16-token
    pieces, heads that do not fill the matrix columns, and an infinite value or a NaN score in the tail, as in 64 bits."""
    sh = hb.make_shape(B, G * Hkv, Hkv, 64 * T, dtype=torch.float16 if dtype == "fp16" else torch.bfloat16)
    dt, lens = hb.torch_dtype(sh), [0, 1, 15, 16, 17, 63, 64]
    g = torch.Generator(device="cuda").manual_seed(70 + T)
    K, V = (torch.randn((B, Hkv, 64 * T, 128), device="cuda", generator=g).to(dt) for _ in range(2))
    tk, tv = (torch.randn((B, Hkv, 64, 128), device="cuda", generator=g).to(dt) for _ in range(2))
    Q = torch.randn((B, G * Hkv, 128), device="cuda", generator=g).to(dt)
    for b, n in enumerate(lens):                      # tokens past a row's tail must not be looked at
        tk[b, :, n:], tv[b, :, n:] = float("nan"), float("inf")
    tv[5, -1, 62, 7], tv[6, -1, 3, 127], tk[4, 0, 16, 9] = float("inf"), float("-inf"), float("nan")
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K, V)
    Ku, Vu = hb.unpack_kv(sh, kv)
    O, LSE = hb.decode_attn(sh, Q, kv, tail_k=tk, tail_v=tv, tail_len=torch.tensor(lens, dtype=torch.int32, device="cuda"))
    O, LSE = O.double().cpu(), LSE.double().cpu()
    for b, n in enumerate(lens):
        for h in range(Hkv):
            k, v, q = (x.double().cpu() for x in (torch.cat([Ku[b, h], tk[b, h, :n]]), torch.cat([Vu[b, h], tv[b, h, :n]]), Q[b, h * G:(h + 1) * G]))
            S = q @ k.T * 128 ** -0.5
            Or, Lr = (torch.softmax(S, 1)[:, :, None] * v).sum(1), torch.logsumexp(S, 1)
            got, lse = O[b, h * G:(h + 1) * G], LSE[b, h * G:(h + 1) * G]
            fin = torch.isfinite(Or)
            assert torch.equal(torch.isnan(got), torch.isnan(Or)) and torch.equal(got[torch.isinf(Or)], Or[torch.isinf(Or)]), (b, h)
            assert torch.equal(torch.isnan(lse), torch.isnan(Lr)), (b, h)
            if fin.any():
                assert_close(got[fin].numpy(), Or[fin].numpy(), f"tail of {n} in row {b}, kv head {h}")
            if torch.isfinite(Lr).all():
                assert_lse_close(lse.numpy(), Lr.numpy(), f"tail of {n} in row {b}, kv head {h} lse")


@pytest.mark.parametrize("B,Hkv,T", [(1, 1, 1), (2, 1, 8), (1, 2, 9), (16, 8, 16), (64, 4, 5), (64, 4, 127), (50, 4, 160)])
@pytest.mark.parametrize("dtype,pol", [("bf16", dict()), ("fp16", dict()), ("bf16", dict(sparse_frac_k=0.0)), ("fp16", dict(sparse_frac_k=0.0, sparse_frac_v=0.0)),
                                       ("bf16", dict(sparse_frac_k=0.5, sparse_frac_v=0.5)), ("fp16", dict(skip_frac=0.5)), ("bf16", "empty")])
def test_decode_rows_served_by_one_workgroup(B, Hkv, T, dtype, pol):
    """Short rows and rows numerous enough: O and LSE written without a merge, wherever O begins; against the
    same call cut into three splits, which is checked against the oracle elsewhere."""
    G = 3
    sh = hb.make_shape(B, G * Hkv, Hkv, 64 * T, dtype=torch.float16 if dtype == "fp16" else torch.bfloat16)
    dt = hb.torch_dtype(sh)
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V = (torch.randn((B, Hkv, 64 * T, 128), device="cuda", generator=g).to(dt) for _ in range(2))
    V[:, :, ::61, 3] = 1e-6                            # bf16: tiles of both encodings
    V[:, :, :64] = V[:, :, :64].clamp(0.1, 1.0)
    if pol == "empty":
        s = np.zeros((B, Hkv, T), dtype=np.int8)
        s[::2] = 2                                     # every other batch row holds nothing
        pol = dict(state_k=s, state_v=s)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K, V)
    Q = torch.randn((B, G * Hkv, 128), device="cuda", generator=g).to(dt)
    O3, L3 = hb.decode_attn(sh, Q, kv, n_splits=3)
    out = torch.empty(Q.numel() + 1, device="cuda", dtype=dt)[1:].view_as(Q)      # 2-byte aligned
    for o in (None, out):
        O, LSE = hb.decode_attn(sh, Q, kv, out=o)
        assert (torch.isneginf(LSE) == torch.isneginf(L3)).all()
        seen = ~torch.isneginf(L3)
        assert (LSE[seen] - L3[seen]).abs().max() < 1e-5 and (O[~seen] == 0).all()
        # fp32 accumulation in another order, then one rounding to 16 bits
        assert (O.float() - O3.float()).abs().max() <= (2 ** -8 if dt is torch.bfloat16 else 2 ** -11) * 1.01 * O3.float().abs().max()


@pytest.mark.parametrize("B,Hkv,T", [(3, 8, 72), (5, 8, 70), (33, 4, 40), (8, 8, 256), (1, 3, 301)])
@pytest.mark.parametrize("pol", [dict(), dict(sparse_frac_k=0.0, sparse_frac_v=0.0), dict(skip_frac=0.5, sparse_frac_k=0.5)])
def test_decode_number_of_splits_is_the_librarys_choice(B, Hkv, T, pol):
    """Row counts that do not divide the compute units: the choice fits the workspace of hs_decode_auto_splits, its
    two phases agree on it, and the result is that of an explicit count."""
    sh = hb.make_shape(B, 2 * Hkv, Hkv, 64 * T)
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V = (torch.randn((B, Hkv, 64 * T, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K, V)
    Q = torch.randn((B, 2 * Hkv, 128), device="cuda", generator=g).bfloat16()
    O2, L2 = hb.decode_attn(sh, Q, kv, n_splits=2)
    n = hb.workspace_bytes(sh, 2, 0)
    for phases in ((3,), (1, 2)):
        ws = torch.full((n + 4096,), 255, dtype=torch.uint8, device="cuda")
        O, LSE = torch.empty_like(Q), torch.empty(Q.shape[:2], device="cuda")
        for ph in phases:
            hb.decode_attn(sh, Q, kv, out=O, lse=LSE, workspace=ws, phases=ph)
        assert (ws[n:] == 255).all()
        assert (LSE - L2).abs().max() < 1e-5
        assert (O.float() - O2.float()).abs().max() <= 2 ** -8 * 1.01 * O2.float().abs().max()


@pytest.mark.parametrize("B,Hkv,T", [(1, 1, 4), (16, 8, 16), (64, 4, 100),                      # one workgroup per row
                                     (3, 8, 72), (5, 8, 70), (33, 4, 40), (8, 8, 256), (1, 3, 301)])   # the library's split count
@pytest.mark.parametrize("dtype,pol", [("bf16", dict()), ("fp16", dict(sparse_frac_k=0.0, sparse_frac_v=0.0)),
                                       ("bf16", dict(skip_frac=0.5, sparse_frac_k=0.5)), ("fp16", "empty")])
def test_decode_default_call_against_64_bits(B, Hkv, T, dtype, pol):
    """What the library chooses by itself, against fp64 attention over the unpacked cache (whose bytes the oracle pins)."""
    G = 3
    sh = hb.make_shape(B, G * Hkv, Hkv, 64 * T, dtype=torch.float16 if dtype == "fp16" else torch.bfloat16)
    dt = hb.torch_dtype(sh)
    g = torch.Generator(device="cuda").manual_seed(60 + T)
    K, V = (torch.randn((B, Hkv, 64 * T, 128), device="cuda", generator=g).to(dt) for _ in range(2))
    if pol == "empty":
        s = np.full((B, Hkv, T), 2, dtype=np.int8)
        s[::3, 0] = 0                                  # rows that hold nothing
        s[:, :, 1::2] = 0
        pol = dict(state_k=s, state_v=s)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K, V)
    del K, V
    Q = torch.randn((B, G * Hkv, 128), device="cuda", generator=g).to(dt)
    O, LSE = hb.decode_attn(sh, Q, kv)
    Ku, Vu = hb.unpack_kv(sh, kv)
    seen = (kv.k_map != 0).repeat_interleave(64, -1)
    Or, Lr = torch.zeros(B, G * Hkv, 128, dtype=torch.float64), torch.full((B, G * Hkv), -np.inf, dtype=torch.float64)
    for b in range(B):
        for h in range(Hkv):
            k, v, q = (x.double() for x in (Ku[b, h][seen[b, h]], Vu[b, h][seen[b, h]], Q[b, h * G:(h + 1) * G]))
            if len(k):
                S = q @ k.T * 128 ** -0.5
                Or[b, h * G:(h + 1) * G], Lr[b, h * G:(h + 1) * G] = (torch.softmax(S, 1) @ v).cpu(), torch.logsumexp(S, 1).cpu()
    assert_lse_close(LSE.cpu().numpy(), Lr.numpy(), "decode default call lse")
    assert_close(_f32(O), Or.numpy(), "decode default call")


@pytest.mark.parametrize("B,Hkv,T,counts,n", [
    (8, 8, 512, None, 4), (3, 8, 512, None, 10), (1, 8, 1024, None, 32), (4, 8, 512, None, 8),     # room for any states
    (8, 8, 640, [0, 0, 640, 0, 640], 4),                                                           # a slot per tile, no promise
    (8, 8, 512, [0, 128, 384, 128, 384], 3), (8, 8, 512, [128, 128, 256, 0, 384], 4)])             # fractions: nothing / a quarter skipped
def test_decode_splits_of_caches_whose_fill_the_host_does_not_know(B, Hkv, T, counts, n):
    """Pools with room beyond what a policy's fractions keep (states on the device, growing caches) do not count as full:
    their rows get as many splits as fit the chip.  Counted by the partials that the split kernel writes."""
    sh = hb.make_shape(B, Hkv, Hkv, 64 * T)
    kv = hb.PackedKV(sh, counts or [0, T, T, T, T])
    kv.uniform = 0
    kv.k_map.zero_(), kv.v_map.zero_()                 # nothing kept: the pools are not looked at
    Q = torch.randn((B, Hkv, 128), device="cuda").bfloat16()
    ws = torch.full((hb.workspace_bytes(sh, 2, 0),), 255, dtype=torch.uint8, device="cuda")
    hb.decode_attn(sh, Q, kv, workspace=ws, phases=1)
    assert int((ws.view(torch.int32) != -1).sum()) == B * Hkv * 129 * n


def test_decode_tail_of_a_batch_beyond_one_grid():
    """40000 rows of one tile: the tail's planes of the grid no longer fit behind the rows' own."""
    B, L = 40000, 64
    sh = hb.make_shape(B, 1, 1, L)
    g = torch.Generator(device="cuda").manual_seed(3)
    K, V, tk, tv = (torch.randn((B, 1, L, 128), device="cuda", generator=g).bfloat16() for _ in range(4))
    Q = torch.randn((B, 1, 128), device="cuda", generator=g).bfloat16()
    kv = hb.compress_kv(sh, hb.make_policy(sparse_frac_k=0.0, sparse_frac_v=0.0), K, V)
    O, LSE = hb.decode_attn(sh, Q, kv, tail_k=tk, tail_v=tv, tail_len=33)
    pick = torch.tensor([0, 1, 25534, 25535, 32767, 39999], device="cuda")
    k, v = torch.cat([K[pick, 0], tk[pick, 0, :33]], 1).double(), torch.cat([V[pick, 0], tv[pick, 0, :33]], 1).double()
    s = (k * Q[pick].double()).sum(-1) * 128 ** -0.5
    assert_lse_close(LSE[pick, 0].cpu().numpy(), torch.logsumexp(s, 1).cpu().numpy(), "tail of a large batch lse")
    assert_close(_f32(O[pick, 0]), (torch.softmax(s, 1)[:, :, None] * v).sum(1).cpu().numpy(), "tail of a large batch")


def _nan_case(T, Lq, dtype, seed):
    """Two kv heads of two query heads.  kv head 0 holds one NaN key; of kv head 1's queries every third of head 2 is NaN and
    (bf16) head 3 meets a tile in which every score is -inf.  Q, K, V as torch tensors on the CPU and the NaN key's token."""
    L, dt = 64 * T, torch.float16 if dtype == "fp16" else torch.bfloat16
    g = torch.Generator().manual_seed(seed)
    Q, K, V = (torch.randn((1, n, m, 128), generator=g).to(dt) for n, m in ((4, Lq), (2, L), (2, L)))
    tok = L - Lq // 2 - 1
    K[0, 0, tok, 9] = float("nan")
    Q[0, 2, ::3, 17] = float("nan")
    if dtype == "bf16":
        K[0, 1, :, 0] = 0
        K[0, 1, 64:128, 0] = -1e30
        Q[0, 2, :, 0], Q[0, 3, :, 0] = 0, 1e30
    return Q, K, V, tok


def _nan_reference(Q, K, V, visible):
    """fp64 attention of Q [4, n, 128] over K, V [2, L, 128]; visible [n, L]."""
    S = torch.matmul(Q.double(), K.double().repeat_interleave(2, 0).transpose(1, 2)) * 128 ** -0.5
    S = torch.where(S < -1e30, float("-inf"), S).masked_fill(~visible, float("-inf"))    # beyond what fp32 holds
    lse = torch.logsumexp(S, -1)
    return torch.matmul(torch.softmax(S, -1), V.double().repeat_interleave(2, 0)), lse


def _check_nan_rows(O, LSE, Or, Lr, what):
    nan = torch.isnan(Lr)
    assert nan.any() and (~nan).any()
    assert torch.isnan(LSE[nan]).all() and torch.isnan(O[nan].float()).all(), what
    assert_close(_f32(O[~nan]), Or[~nan].numpy(), what)
    assert_lse_close(LSE[~nan].numpy(), Lr[~nan].numpy(), what)


@pytest.mark.parametrize("dtype,pol", [("bf16", dict()), ("fp16", dict(sparse_frac_k=0.0)), ("bf16", dict(sparse_frac_k=0.0, sparse_frac_v=0.0)),
                                       ("fp16", dict()), ("bf16", dict(sparse_frac_v=0.0)), ("bf16", dict(dense_first_tiles=1, dense_last_tiles=4)),
                                       ("fp16", dict(sparse_frac_k=0.5))])
def test_prefill_nan_scores_come_out_however_the_tiles_are_cut(dtype, pol):
    """A query that sees a NaN score has O and LSE NaN, in one range and in several; the others see nothing of it."""
    import ctypes as C
    T, Lq = 70, 128
    Q, K, V, tok = _nan_case(T, Lq, dtype, 970)
    sh = hb.make_shape(1, 4, 2, 64 * T, dtype=Q.dtype)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K.cuda(), V.cuda())
    Ku, Vu = (t.cpu()[0] for t in hb.unpack_kv(sh, kv))
    at = 64 * T - Lq
    Or, Lr = _nan_reference(Q[0], Ku, Vu, torch.arange(64 * T) <= at + torch.arange(Lq)[:, None])
    Qd, kvs, one = Q.cuda(), kv.struct(), 4 * Lq * 129 * 4
    assert hb.prefill_workspace_bytes(sh, Lq, at, kv) >= 5 * one
    ws = torch.empty(5 * one, dtype=torch.uint8, device="cuda")
    for n in (1, 2, 5):
        O, LSE = torch.zeros_like(Qd), torch.zeros(Qd.shape[:3], device="cuda")
        hb._check(hb.lib().hs_prefill_attn_ws(C.byref(sh), Lq, at, 0.0, 1, hb._ptr(Qd), C.byref(kvs), hb._ptr(O), hb._ptr(LSE), hb._ptr(ws),
                                              n * one, hb._stream()))
        _check_nan_rows(O.cpu()[0], LSE.cpu()[0], Or, Lr, f"prefill with NaN scores in {n} ranges")
        for slab in (16, 32):
            O, LSE = hb.prefill_attn_planned(sh, Qd, kv, slab, n)
            _check_nan_rows(O.cpu()[0], LSE.cpu()[0], Or, Lr, f"prefill with NaN scores in {n} ranges, slabs of {slab}")


@pytest.mark.parametrize("T", [6, 70])
@pytest.mark.parametrize("dtype,pol", [("bf16", dict()), ("fp16", dict(sparse_frac_k=0.0)), ("bf16", dict(sparse_frac_k=0.0, sparse_frac_v=0.0))])
def test_decode_nan_scores_come_out_however_the_tiles_are_split(T, dtype, pol):
    Q, K, V, tok = _nan_case(T, 2, dtype, 980)
    q = Q[:, :, 0].contiguous()
    sh = hb.make_shape(1, 4, 2, 64 * T, dtype=Q.dtype)
    kv = hb.compress_kv(sh, hb.make_policy(**pol), K.cuda(), V.cuda())
    Ku, Vu = (t.cpu()[0] for t in hb.unpack_kv(sh, kv))
    Or, Lr = _nan_reference(q[0][:, None], Ku, Vu, torch.ones(1, 64 * T, dtype=torch.bool))
    for n in (1, 2, 5, 0):
        O, LSE = hb.decode_attn(sh, q.cuda(), kv, n_splits=n)
        _check_nan_rows(O.cpu()[0][:, None], LSE.cpu()[0][:, None], Or, Lr, f"decode with NaN scores, {n} splits")
    # the same tokens again as a dense tail that follows a cache without them
    tk, tv = torch.zeros(1, 2, 64, 128, dtype=Q.dtype), torch.zeros(1, 2, 64, 128, dtype=Q.dtype)
    tk[:, :, :20], tv[:, :, :20] = K[:, :, tok - 19:tok + 1], V[:, :, tok - 19:tok + 1]
    clean = K.clone()
    clean[0, 0, tok, 9] = 1.0
    kv = hb.compress_kv(sh, hb.make_policy(**pol), clean.cuda(), V.cuda())
    Ku, Vu = (t.cpu()[0] for t in hb.unpack_kv(sh, kv))
    Or, Lr = _nan_reference(q[0][:, None], torch.cat([Ku, tk[0, :, :20]], 1), torch.cat([Vu, tv[0, :, :20]], 1), torch.ones(1, 64 * T + 20, dtype=torch.bool))
    O, LSE = hb.decode_attn(sh, q.cuda(), kv, tail_k=tk.cuda(), tail_v=tv.cuda(), tail_len=20)
    _check_nan_rows(O.cpu()[0][:, None], LSE.cpu()[0][:, None], Or, Lr, "decode with NaN scores in the tail")


def test_append_tiles_during_decode():
    """A cache allocated for 9 tiles, compressed with 4, then grown tile by tile (mixed tile kinds, the last
    one from a strided buffer); after every append decode equals the oracle's, and at the end pools and maps
    are those of compressing everything at once."""
    B, Hq, Hkv, L = 2, 8, 2, 64 * 9
    T = L // 64
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=170)
    q = Q[:, :, 0, :].copy()
    rng = np.random.default_rng(171)
    sk = rng.choice([1, 2], size=(T,)).astype(np.int8)
    sv = rng.choice([1, 2], size=(T,)).astype(np.int8)
    full_k, full_v = np.broadcast_to(sk, (B, Hkv, T)).copy(), np.broadcast_to(sv, (B, Hkv, T)).copy()
    pre_k, pre_v = full_k.copy(), full_v.copy()
    pre_k[:, :, 4:] = 0
    pre_v[:, :, 4:] = 0
    sh = hb.make_shape(B, Hq, Hkv, L)
    caps = [0, int((sk == 1).sum()), int((sk == 2).sum()), int((sv == 1).sum()), int((sv == 2).sum())]
    kv = hb.PackedKV(sh, caps)
    hb.compress_kv(sh, hb.make_policy(state_k=pre_k, state_v=pre_v), _dev(K), _dev(V), out=kv)
    pk, pv, _ = orc.compress_kv(K, V, state_k=pre_k, state_v=pre_v)
    ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
    Kd, Vd = _dev(K), _dev(V)
    for t in range(4, T):
        kt, vt = Kd[:, :, 64 * t:64 * (t + 1)], Vd[:, :, 64 * t:64 * (t + 1)]      # strided views of the full tensors
        if t % 2 == 0:
            kt, vt = kt.contiguous(), vt.contiguous()
        hb.append_tile(sh, kv, t, kt, vt, state_k=int(sk[t]), state_v=int(sv[t]), overflow=ovf)
        orc.append_tile(pk, pv, t, K[:, :, 64 * t:64 * (t + 1)], V[:, :, 64 * t:64 * (t + 1)], int(sk[t]), int(sv[t]))
        O, LSE = hb.decode_attn(sh, _dev(q), kv)
        torch.cuda.synchronize()
        Or, Lr = orc.attention_decode(q, pk, pv)
        assert_close(_f32(O), Or, f"decode after append of tile {t}")
        assert_lse_close(LSE.cpu().numpy(), Lr, f"decode after append of tile {t} lse")
    assert int(ovf.item()) == 0
    pk1, pv1, _ = orc.compress_kv(K, V, state_k=full_k, state_v=full_v)
    check_packed_bit_exact(sh, kv, pk1, pv1)
    # a full pool: the tile stays skipped and the flag goes up
    kv2 = hb.PackedKV(sh, [0, 1, 4, 1, 4])
    z = np.zeros((B, Hkv, T), dtype=np.int8)
    z[:, :, :4] = 2
    hb.compress_kv(sh, hb.make_policy(state_k=z, state_v=z), Kd, Vd, out=kv2)
    hb.append_tile(sh, kv2, 4, Kd[:, :, 256:320].contiguous(), Vd[:, :, 256:320].contiguous(), overflow=ovf)
    torch.cuda.synchronize()
    assert int(ovf.item()) == 1
    assert (kv2.k_map[:, :, 4].cpu().numpy() == 0).all() and (kv2.v_map[:, :, 4].cpu().numpy() == 0).all()
    import ctypes as C
    kvs = kv2.struct()
    args = (hb._ptr(Kd), hb._ptr(Vd), None, C.byref(kvs), None, None)
    assert hb.lib().hs_append_tile(C.byref(sh), T, 2, 2, 0, *args) == -1          # tile out of range
    assert hb.lib().hs_append_tile(C.byref(sh), 5, 0, 2, 0, *args) == -1          # SKIP is not a state to append
    assert hb.lib().hs_append_tile(C.byref(sh), 5, 2, 2, 7, *args) == -1          # unknown element rule


@pytest.mark.parametrize("T,n,rows", [(5, 2, 2), (300, 64, 2), (300, 63, 3), (2100, 1000, 2), (1100, 500, 8)])   # both ways of counting
@pytest.mark.parametrize("state_k,state_v", [(2, 2), (1, 2)])
def test_append_counts_what_the_row_holds(T, n, rows, state_k, state_v):
    """New tiles take the slots after those their row holds, wherever they stand and whatever their old entries are;
    tiles that find a pool full stay SKIP and raise the flag."""
    rng = np.random.default_rng(T + n)
    at = T // 3
    sk, sv = rng.integers(1, 3, (1, rows, T)).astype(np.int8), rng.integers(1, 3, (1, rows, T)).astype(np.int8)
    hole = rng.random((1, rows, T)) < 0.3
    sk[hole], sv[hole] = 0, 0
    sk[:, :, at:at + n], sv[:, :, at:at + n] = 0, 0
    held = [int(((s == k).sum(-1)).max()) for s, k in ((sk, 1), (sk, 2), (sv, 1), (sv, 2))]
    room = n - 1                                      # one tile too few in the fullest row's pools
    caps = [0, held[0] + room * (state_k == 1), held[1] + room * (state_k == 2), held[2] + room * (state_v == 1), held[3] + room * (state_v == 2)]
    sh = hb.make_shape(1, rows, rows, 64 * T)
    kv = hb.PackedKV(sh, caps)
    kv.uniform = 0
    maps = [np.zeros((1, rows, T), dtype=np.int32) for _ in range(2)]
    for m, s in zip(maps, (sk, sv)):
        for r in range(rows):
            for state, sign in ((1, 1), (2, -1)):
                idx = np.flatnonzero(s[0, r] == state)
                m[0, r, idx] = sign * (np.arange(len(idx)) + 1)
    kv.k_map.copy_(torch.from_numpy(maps[0]))
    kv.v_map.copy_(torch.from_numpy(maps[1]))
    g = torch.Generator(device="cuda").manual_seed(T)
    K = torch.randn((1, rows, 64 * n, 128), device="cuda", generator=g).bfloat16()
    V = torch.randn((1, rows, 64 * n, 128), device="cuda", generator=g).bfloat16()
    for _ in range(2):                                # a second call over the same place gives the same again
        over = torch.zeros(1, dtype=torch.int32, device="cuda")
        hb.append_tile(sh, kv, at, K, V, state_k=state_k, state_v=state_v, overflow=over)
        km, vm = lib_maps(kv.k_map, kv.v_map)[:2]
        want = [m.copy() for m in maps]
        full = False
        for r in range(rows):
            ck, cv = int((sk[0, r] == state_k).sum()), int((sv[0, r] == state_v).sum())
            for i in range(n):
                if ck + i < caps[state_k] and cv + i < caps[2 + state_v]:
                    want[0][0, r, at + i] = (ck + i + 1) * (1 if state_k == 1 else -1)
                    want[1][0, r, at + i] = (cv + i + 1) * (1 if state_v == 1 else -1)
                else:
                    full = True
        assert (km == want[0]).all() and (vm == want[1]).all()
        assert int(over.item()) == int(full)


def _pool_bytes_equal(a, b):
    for name in ("k_dense", "k_nnz", "k_meta", "v_dense", "v_nnz", "v_meta", "k_map", "v_map"):
        x, y = getattr(a, name), getattr(b, name)
        assert (x is None) == (y is None) and (x is None or torch.equal(x, y)), name


@pytest.mark.parametrize("T,B", [(4, 260), (17, 60), (33, 20), (64, 5)])
@pytest.mark.parametrize("pol", [dict(skip_frac=0.5), dict(sparse_frac_k=0.5), dict(skip_frac=0.25, sparse_frac_k=0.3, sparse_frac_v=0.7), dict(sparse_frac_k=0.0, sparse_frac_v=0.6),
                                 dict(skip_frac=0.9, sparse_frac_k=0.5, dense_first_tiles=1, dense_last_tiles=4), dict(skip_frac=0.4, dense_first_tiles=70),
                                 dict(skip_frac=0.3, sparse_frac_v=0.2, element_rule=1)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_short_rows_ranked_by_the_pack_kernel_give_the_same_bytes(T, B, pol, dtype):
    """Rows ranked by the selection kernel (a batch of them) and by the pack kernel itself (one sequence at a time), with
    scores that tie inside a row and rows that hold nothing but zeros."""
    Hkv, L = 2, 64 * T
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V = (torch.randn((B, Hkv, L, 128), device="cuda", generator=g).to(dtype) for _ in range(2))
    for x in (K, V):
        y = x.view(B, Hkv, T, 64, 128)
        y[:, :, 3::4] = y[:, :, 1:2]                  # equal tiles
        y[1, 0] = 0
        y[2, 1, ::2] = 0
    names = ("k_dense", "k_nnz", "k_meta", "v_dense", "v_nnz", "v_meta", "k_map", "v_map")

    def packed(k, v):
        sh = hb.make_shape(len(k), Hkv, Hkv, L, dtype=dtype)
        kv = hb.compress_kv(sh, hb.make_policy(**pol), k, v)
        return [None if getattr(kv, n) is None else getattr(kv, n).reshape(len(k), -1) for n in names]
    many = packed(K, V)
    for b in range(0, B, 3):
        for x, y, n in zip(many, packed(K[b:b + 1], V[b:b + 1]), names):
            assert (x is None) == (y is None) and (x is None or torch.equal(x[b:b + 1], y)), (b, n)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("state_k,state_v", [(2, 2), (1, 2), (2, 1), (1, 1)])
@pytest.mark.parametrize("rule,places", [(0, "rows"), (1, "rows"), (0, 3), (1, 300)])
def test_append_of_few_tiles_and_of_many_write_the_same_bytes(dtype, state_k, state_v, rule, places):
    """520 rows in one call and in calls of fewer rows, which take a workgroup of 8 waves per tile: places per row (some rows left
    out, some pools full) or one for all, tokens and heads in an order of their own, values that fp16 does not hold."""
    B, Hkv, T = 65, 8, 310
    g = torch.Generator(device="cuda").manual_seed(31)
    K, V = (torch.randn((B, 64, Hkv, 136), device="cuda", generator=g).to(dtype)[..., :128].transpose(1, 2) for _ in range(2))
    K, V = (torch.where(torch.rand(x.shape, device="cuda", generator=g) < 0.6, x, torch.zeros_like(x)) for x in (K, V)) if rule else (K, V)
    K, V = (torch.empty((B, 64, Hkv, 136), device="cuda", dtype=dtype)[..., :128].transpose(1, 2).copy_(x) for x in (K, V))
    if dtype == torch.bfloat16:
        V[::5, :, 9, 3] = 1e-30
    maps = torch.zeros((B, Hkv, T), dtype=torch.int32)
    held = torch.randint(0, 5, (B,), generator=torch.Generator().manual_seed(32))
    for b in range(B):
        maps[b, :, 5:5 + held[b]] = -torch.arange(1, held[b] + 1, dtype=torch.int32)
        maps[b, :, 290:290 + held[b]] = torch.arange(1, held[b] + 1, dtype=torch.int32)
    at = torch.randint(-1, 5, (B,), generator=torch.Generator().manual_seed(33), dtype=torch.int32)
    at[held == 1] = 309
    results = []
    for parts in ((slice(0, B),), (slice(0, 1), slice(1, 64), slice(64, B))):
        out = []
        for p in parts:
            n = len(range(B)[p])
            sh = hb.make_shape(n, Hkv, Hkv, 64 * T, dtype=dtype)
            kv = hb.PackedKV(sh, [0, 4, 4, 4, 4])     # rows that hold four of a kind are full
            kv.uniform = 0
            for x in (kv.k_dense, kv.k_nnz, kv.k_meta, kv.v_dense, kv.v_nnz, kv.v_meta):
                x.fill_(7)
            kv.k_map.copy_(maps[p]), kv.v_map.copy_(maps[p])
            over = torch.zeros(1, dtype=torch.int32, device="cuda")
            hb.append_tile(sh, kv, at[p].cuda() if places == "rows" else places, K[p], V[p], state_k, state_v, element_rule=rule, overflow=over)
            out.append([x.cpu().reshape(n, -1) for x in (kv.k_dense, kv.k_nnz, kv.k_meta, kv.v_dense, kv.v_nnz, kv.v_meta, kv.k_map, kv.v_map)] + [over.cpu()])
        results.append([torch.cat([o[i] for o in out]) for i in range(8)] + [max(int(o[8]) for o in out)])
    many, few = results
    assert many[8] == few[8] == 1
    for i in range(8):
        assert torch.equal(many[i], few[i]), i


@pytest.mark.parametrize("state_k,state_v", [(2, 2), (1, 2)])
def test_append_beyond_the_last_level_cache_in_one_launch(state_k, state_v):
    """More than 256 MB of new K and V (read non-temporally) that one launch still counts: the bytes of shorter calls."""
    B, Hkv, n, T = 16, 8, 64, 80                       # 128 rows x 64 tiles; 64 x 128 x 80 entries to count
    sh = hb.make_shape(B, Hkv, Hkv, 64 * T)
    g = torch.Generator(device="cuda").manual_seed(21)
    K, V = (torch.randn((B, Hkv, 64 * n, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    got = []
    for step in (n, 16):
        kv = hb.PackedKV(sh, [0] + [n * (state_k == 1), n * (state_k == 2), n * (state_v == 1), n * (state_v == 2)])
        kv.uniform = 0
        for t in (kv.k_dense, kv.k_nnz, kv.k_meta, kv.v_dense, kv.v_nnz, kv.v_meta, kv.k_map, kv.v_map):
            if t is not None:
                t.zero_()
        over = torch.zeros(1, dtype=torch.int32, device="cuda")
        for i in range(0, n, step):
            part = slice(64 * i, 64 * (i + step))
            hb.append_tile(sh, kv, 5 + i, K[:, :, part], V[:, :, part], state_k=state_k, state_v=state_v, overflow=over)
        assert int(over.item()) == 0
        got.append(kv)
    _pool_bytes_equal(*got)


def test_append_of_one_tile_to_many_rows_beyond_the_last_level_cache():
    """The same by a tile index per batch row: 8000 rows, against a compression of each half."""
    B, Hkv = 1000, 8
    sh, half = hb.make_shape(B, Hkv, Hkv, 64), hb.make_shape(B // 2, Hkv, Hkv, 64)
    g = torch.Generator(device="cuda").manual_seed(22)
    K, V = (torch.randn((B, Hkv, 64, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    kv = hb.PackedKV(sh, [0, 0, 1, 0, 1])
    kv.uniform = 0
    kv.k_map.zero_(), kv.v_map.zero_()
    hb.append_tile(sh, kv, torch.zeros(B, dtype=torch.int32, device="cuda"), K, V)
    parts = [hb.compress_kv(half, hb.make_policy(), K[i:i + B // 2], V[i:i + B // 2]) for i in (0, B // 2)]
    for name in ("k_nnz", "k_meta", "v_nnz", "v_meta", "k_map", "v_map"):
        assert torch.equal(getattr(kv, name), torch.cat([getattr(p, name) for p in parts])), name


@pytest.mark.parametrize("n_splits", [2, 4, 6, 8, 12, 16])
@pytest.mark.parametrize("B,Hkv,dense", [(3, 3, False), (7, 1, True), (2, 8, False)])
def test_splits_of_rows_that_may_differ_start_further_on_from_row_to_row(n_splits, B, Hkv, dense):
    """Every split of every row is worked on once, whatever the row it starts at: rows of different length, one of them empty,
    even numbers of splits with every power of two in them, more and fewer than the rows have tiles."""
    G, T = 2, 19
    L = 64 * T
    Q, K, V = wl.make_qkv(B, G * Hkv, Hkv, L, 128, 1, seed=1230 + B)
    q = Q[:, :, 0, :].copy()
    sk = np.full((B, Hkv, T), orc.DENSE if dense else orc.SPARSE24, dtype=np.int8)
    sv = np.full((B, Hkv, T), orc.SPARSE24, dtype=np.int8)
    for i in range(B * Hkv):
        held = (7 * i) % (T + 1)
        sk.reshape(-1, T)[i, held:] = 0
        sv.reshape(-1, T)[i, held:] = 0
    sh = hb.make_shape(B, G * Hkv, Hkv, L)
    kv = hb.compress_kv(sh, hb.make_policy(state_k=sk, state_v=sv), _dev(K), _dev(V), out=hb.PackedKV(sh, [0, T, T, T, T]))
    pk, pv, _ = orc.compress_kv(K, V, state_k=sk, state_v=sv)
    _, tk, tv = wl.make_qkv(B, G * Hkv, Hkv, 64, 128, 1, seed=1231)
    for tail in (None, np.arange(1, B + 1, dtype=np.int32)):
        kw = {} if tail is None else dict(tail_k=_dev(tk), tail_v=_dev(tv), tail_len=torch.from_numpy(tail).cuda())
        O, LSE = hb.decode_attn(sh, _dev(q), kv, n_splits=n_splits, **kw)
        torch.cuda.synchronize()
        Or, Lr = orc.attention_decode(q, pk, pv, **({} if tail is None else dict(tail_k=tk, tail_v=tv, tail_len=tail)))
        assert_close(_f32(O), Or, f"{n_splits} splits of rows that differ")
        assert_lse_close(LSE.cpu().numpy(), Lr, f"{n_splits} splits of rows that differ lse")


def test_batch_rows_of_different_length_decode_and_append():
    """A batch whose sequences hold 3, 9 and 6 tiles and 17, 0 and 64 tail tokens: decode with one tail
    length per batch row; the row with the full tail (and only that one) appends it at its own position;
    decode again.  Against the oracle throughout, packed state bit for bit."""
    B, Hq, Hkv, T = 3, 8, 2, 10
    L = 64 * T
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=270, k_outliers=True)
    q = Q[:, :, 0, :].copy()
    held = [3, 9, 6]
    sk = np.full((B, Hkv, T), orc.DENSE, dtype=np.int8)
    sv = np.full((B, Hkv, T), orc.SPARSE24, dtype=np.int8)
    for b in range(B):
        sk[b, :, held[b]:] = 0
        sv[b, :, held[b]:] = 0
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv = hb.PackedKV(sh, [0, T, 0, 0, T])
    kv.uniform = 0
    hb.compress_kv(sh, hb.make_policy(state_k=sk, state_v=sv), _dev(K), _dev(V), out=kv)
    pk, pv, _ = orc.compress_kv(K, V, state_k=sk, state_v=sv)
    _, tk, tv = wl.make_qkv(B, Hq, Hkv, 64, 128, 1, seed=271)
    lens = np.array([17, 0, 64], dtype=np.int32)
    lens_d = torch.from_numpy(lens).cuda()
    O, LSE = hb.decode_attn(sh, _dev(q), kv, tail_k=_dev(tk), tail_v=_dev(tv), tail_len=lens_d, n_splits=2)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, pk, pv, tail_k=tk, tail_v=tv, tail_len=lens)
    for b in range(B):
        assert_close(_f32(O)[b], Or[b], f"decode ragged batch row {b}")
    assert_lse_close(LSE.cpu().numpy(), Lr, "decode ragged batch lse")
    where = np.array([-1, -1, held[2]], dtype=np.int32)
    ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
    hb.append_tile(sh, kv, torch.from_numpy(where).cuda(), _dev(tk), _dev(tv), state_k=hb.DENSE, state_v=hb.SPARSE24, overflow=ovf)
    orc.append_tile(pk, pv, where, tk, tv, orc.DENSE, orc.SPARSE24)
    torch.cuda.synchronize()
    assert int(ovf.item()) == 0
    check_packed_bit_exact(sh, kv, pk, pv)
    lens2 = np.array([18, 1, 0], dtype=np.int32)            # one more token each; row 2 starts a new tail
    O, LSE = hb.decode_attn(sh, _dev(q), kv, tail_k=_dev(tk), tail_v=_dev(tv), tail_len=torch.from_numpy(lens2).cuda())
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, pk, pv, tail_k=tk, tail_v=tv, tail_len=lens2)
    for b in range(B):
        assert_close(_f32(O)[b], Or[b], f"decode ragged batch after append row {b}")
    assert_lse_close(LSE.cpu().numpy(), Lr, "decode ragged batch after append lse")


def test_serving_loop_two_sequences_of_different_length():
    """The calls in the order a serving loop issues them, for a batch of two sequences of different length:
    compress the whole tiles of each prompt (keys dense, values 2:4), prune the keys further for decode,
    then 70 decode steps in which every new token goes to the dense tail and a full tail moves into the
    cache of its own sequence.  Oracle state and outputs are checked along the way."""
    B, Hq, Hkv, T = 2, 8, 2, 8
    L = 64 * T
    prompt = [64 * 5 + 17, 64 * 3 + 40]
    steps = 70
    total = max(prompt) + steps
    rng = np.random.default_rng(280)
    Kall = wl.f32_to_bf16_bits(rng.standard_normal((B, Hkv, total, 128)).astype(np.float32))
    Vall = wl.f32_to_bf16_bits(rng.standard_normal((B, Hkv, total, 128)).astype(np.float32))
    Qall = wl.f32_to_bf16_bits(rng.standard_normal((B, Hq, steps, 128)).astype(np.float32))
    held = [p // 64 for p in prompt]
    tail_n = [p % 64 for p in prompt]
    K0, V0 = np.zeros((B, Hkv, L, 128), dtype=np.uint16), np.zeros((B, Hkv, L, 128), dtype=np.uint16)
    sk, sv = np.zeros((B, Hkv, T), dtype=np.int8), np.zeros((B, Hkv, T), dtype=np.int8)
    tk, tv = np.zeros((B, Hkv, 64, 128), dtype=np.uint16), np.zeros((B, Hkv, 64, 128), dtype=np.uint16)
    for b in range(B):
        n = 64 * held[b]
        K0[b, :, :n], V0[b, :, :n] = Kall[b, :, :n], Vall[b, :, :n]
        sk[b, :, :held[b]], sv[b, :, :held[b]] = orc.DENSE, orc.SPARSE24
        tk[b, :, :tail_n[b]], tv[b, :, :tail_n[b]] = Kall[b, :, n:prompt[b]], Vall[b, :, n:prompt[b]]
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv_prefill = hb.PackedKV(sh, [0, T, 0, 0, T])
    kv_prefill.uniform = 0
    hb.compress_kv(sh, hb.make_policy(state_k=sk, state_v=sv), _dev(K0), _dev(V0), out=kv_prefill)
    pk, pv, _ = orc.compress_kv(K0, V0, state_k=sk, state_v=sv)
    # decode policy: every key tile 2:4 as well
    kv = hb.recompress_kv(sh, kv_prefill, hb.make_policy(), counts=[0, 0, T, 0, T])
    pk, pv = orc.recompress_kv(pk, pv, np.where(sk == 0, 0, 2), np.where(sv == 0, 0, 2))
    torch.cuda.synchronize()
    check_packed_bit_exact(sh, kv, pk, pv)
    tk_d, tv_d = _dev(tk), _dev(tv)
    ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
    pos = list(prompt)
    checked = 0
    for s_ in range(steps):
        for b in range(B):                                   # the new token's K, V join the tail of its sequence
            tk[b, :, tail_n[b]], tv[b, :, tail_n[b]] = Kall[b, :, pos[b]], Vall[b, :, pos[b]]
            tk_d[b, :, tail_n[b]] = _dev(Kall[b, :, pos[b]])
            tv_d[b, :, tail_n[b]] = _dev(Vall[b, :, pos[b]])
            tail_n[b] += 1
            pos[b] += 1
        q = Qall[:, :, s_, :].copy()
        lens = np.array(tail_n, dtype=np.int32)
        O, LSE = hb.decode_attn(sh, _dev(q), kv, tail_k=tk_d, tail_v=tv_d, tail_len=torch.from_numpy(lens).cuda(), n_splits=2)
        if s_ in (0, 23, 24, 46, 47, 48, steps - 1):
            torch.cuda.synchronize()
            Or, Lr = orc.attention_decode(q, pk, pv, tail_k=tk, tail_v=tv, tail_len=lens)
            for b in range(B):
                assert_close(_f32(O)[b], Or[b], f"serving step {s_} sequence {b}")
            assert_lse_close(LSE.cpu().numpy(), Lr, f"serving step {s_} lse")
            checked += 1
        where = np.array([held[b] if tail_n[b] == 64 else -1 for b in range(B)], dtype=np.int32)
        if (where >= 0).any():                               # a full tail becomes the next tile of its sequence
            hb.append_tile(sh, kv, torch.from_numpy(where).cuda(), tk_d, tv_d, state_k=hb.SPARSE24, state_v=hb.SPARSE24, overflow=ovf)
            orc.append_tile(pk, pv, where, tk, tv, orc.SPARSE24, orc.SPARSE24)
            for b in range(B):
                if where[b] >= 0:
                    held[b] += 1
                    tail_n[b] = 0
    torch.cuda.synchronize()
    assert checked == 7 and int(ovf.item()) == 0 and held == [6, 4] and tail_n == [23, 46]
    check_packed_bit_exact(sh, kv, pk, pv)


def test_chunked_prefill_appends_a_chunk_then_attends_from_its_position():
    """Chunked prefill (the paper's long-context runs use chunks): a cache allocated for the whole sequence
    starts empty; each chunk of 3 tiles is appended in one call (keys dense, values 2:4) and its queries attend
    from their position.  Outputs equal the oracle's causal attention over the one-shot cache; the final
    pools equal one-shot compression; a pool that runs out mid-chunk keeps the tiles that fit."""
    B, Hq, Hkv, T, n = 2, 8, 2, 12, 3
    L = 64 * T
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=260, k_outliers=True)
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv = hb.PackedKV(sh, [0, T, 0, 0, T])
    kv.uniform = 0
    kv.k_map.zero_()
    kv.v_map.zero_()
    sk = np.full((B, Hkv, T), orc.DENSE, dtype=np.int8)
    sv = np.full((B, Hkv, T), orc.SPARSE24, dtype=np.int8)
    pk, pv, _ = orc.compress_kv(K, V, state_k=sk, state_v=sv)
    Kd, Vd, Qd = _dev(K), _dev(V), _dev(Q)
    ovf = torch.zeros(1, dtype=torch.int32, device="cuda")
    for c in range(T // n):
        lo, hi = 64 * n * c, 64 * n * (c + 1)
        hb.append_tile(sh, kv, n * c, Kd[:, :, lo:hi], Vd[:, :, lo:hi], state_k=hb.DENSE, state_v=hb.SPARSE24, overflow=ovf)
        O, LSE = hb.prefill_attn(sh, Qd[:, :, lo:hi].contiguous(), kv, q_start=lo)
        torch.cuda.synchronize()
        rows = [(b, h, i) for b in range(B) for h in range(Hq) for i in range(lo, hi, 5)]
        Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True, q_offset=0)
        got = _f32(O)[:, :, ::5].reshape(-1, 128)
        assert_close(got, Or, f"chunk {c}")
        assert_lse_close(LSE.cpu().numpy()[:, :, ::5].reshape(-1), Lr, f"chunk {c} lse")
    assert int(ovf.item()) == 0
    check_packed_bit_exact(sh, kv, pk, pv)
    small = hb.PackedKV(sh, [0, 4, 0, 0, 5])                # room for 4 dense K tiles and 5 2:4 V tiles
    small.uniform = 0
    small.k_map.zero_()
    small.v_map.zero_()
    hb.append_tile(sh, small, 2, Kd[:, :, :64 * 6], Vd[:, :, :64 * 6], state_k=hb.DENSE, state_v=hb.SPARSE24, overflow=ovf)
    torch.cuda.synchronize()
    assert int(ovf.item()) == 1
    assert (small.k_map.cpu().numpy()[0, 0] == [0, 0, 1, 2, 3, 4, 0, 0, 0, 0, 0, 0]).all()
    assert ((np.abs(small.v_map.cpu().numpy()[1, 1]) & ~hb.MAP_F16) == [0, 0, 1, 2, 3, 4, 0, 0, 0, 0, 0, 0]).all()
    import ctypes as C
    kvs = small.struct()
    args = (hb._ptr(Kd), hb._ptr(Vd), None, C.byref(kvs), None, None)
    assert hb.lib().hs_append_tiles(C.byref(sh), 10, 3, 1, 2, 0, *args) == -1      # runs past the capacity
    assert hb.lib().hs_append_tiles(C.byref(sh), 0, 0, 1, 2, 0, *args) == -1


@pytest.mark.parametrize("seed", range(24))
def test_random_shapes_and_policies(seed):
    """Seeded sweep over shapes (batch, heads, GQA group, tiles, query chunk) and policies (fractions with
    ranking, protected end tiles, explicit states, non-zero rule); every stage against the oracle."""
    rng = np.random.default_rng(1000 + seed)
    B = int(rng.integers(1, 4))
    Hkv = int(rng.integers(1, 4))
    G = int(rng.choice([1, 2, 4, 8]))
    Hq = Hkv * G
    T = int(rng.integers(1, 14))
    L = 64 * T
    Tq = int(rng.integers(1, T + 1))
    Lq = 64 * Tq
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, Lq, seed=2000 + seed, k_outliers=bool(rng.integers(0, 2)))
    kind = int(rng.integers(0, 4))
    if kind == 0:
        pol = dict(skip_frac=float(rng.choice([0.0, 0.25, 0.5])), sparse_frac_k=float(rng.choice([0.0, 0.5, 1.0])),
                   sparse_frac_v=float(rng.choice([0.0, 0.3, 1.0])))
    elif kind == 1:
        pol = dict(skip_frac=float(rng.choice([0.0, 0.4])), dense_first_tiles=int(rng.integers(0, 3)),
                   dense_last_tiles=int(rng.integers(0, 5)))
    elif kind == 2:
        sk, sv = _mixed_states(B, Hkv, T, seed=3000 + seed, p_skip=float(rng.choice([0.0, 0.3])))
        pol = dict(state_k=sk, state_v=sv)
    else:
        pol = dict(element_rule="nonzero", sparse_frac_v=float(rng.choice([0.5, 1.0])))
    sh, kv, pk, pv, info = compress_both(B, Hq, Hkv, L, K, V, **pol)
    if "energy" in info:       # ranked: the cut must not sit on a rounding-level near-tie (see test_compress_policy_ranking)
        for key in ("energy", "loss_k", "loss_v"):
            sc = np.sort(info[key], axis=-1)
            gaps = np.diff(sc, axis=-1) / np.maximum(sc[..., 1:], 1e-300)
            assert ((gaps > 1e-12) | (gaps == 0)).all()
    check_packed_bit_exact(sh, kv, pk, pv)
    causal = bool(rng.integers(0, 4))          # mostly causal
    O, LSE = _prefill(sh, _dev(Q), kv, causal=causal)
    n_rows = min(96, B * Hq * Lq)
    flat = rng.choice(B * Hq * Lq, size=n_rows, replace=False)
    rows = [(int(f // (Hq * Lq)), int((f // Lq) % Hq), int(f % Lq)) for f in flat]
    rows.append((B - 1, Hq - 1, Lq - 1))
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=causal)
    idx = tuple(np.array(rows).T)
    what = f"seed {seed}: B{B} Hq{Hq} Hkv{Hkv} L{L} Lq{Lq} causal={causal} {sorted(pol)}"
    torch.cuda.synchronize()
    assert_close(_f32(O)[idx], Or, "prefill " + what)
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "prefill lse " + what)
    q = Q[:, :, -1, :].copy()
    ns = int(rng.choice([0, 1, 5, 40]))
    Od, LSEd = hb.decode_attn(sh, _dev(q), kv, n_splits=ns)
    torch.cuda.synchronize()
    Odr, Ldr = orc.attention_decode(q, pk, pv)
    assert_close(_f32(Od), Odr, f"decode splits {ns} " + what)
    assert_lse_close(LSEd.cpu().numpy(), Ldr, "decode lse " + what)


@pytest.mark.parametrize("seed", range(8))
def test_random_long_rows_decode(seed):
    """Seeded sweep over rows long enough for decode to hand its tiles out by count (and some just under the
    limits, which go by range): random skip patterns, kinds, protected end tiles, split counts, GQA groups."""
    rng = np.random.default_rng(5000 + seed)
    B = int(rng.integers(1, 3))
    Hkv = int(rng.integers(1, 3))
    G = int(rng.choice([1, 2, 4, 8]))
    Hq = Hkv * G
    T = int(rng.integers(120, 1100))
    L = 64 * T
    dtype = "fp16" if seed % 4 == 3 else "bf16"
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=6000 + seed, k_outliers=bool(rng.integers(0, 2)), dtype=dtype)
    kind = int(rng.integers(0, 3))
    if kind == 0:
        pol = dict(skip_frac=float(rng.choice([0.1, 0.5, 0.9])))
    elif kind == 1:
        pol = dict(skip_frac=float(rng.choice([0.0, 0.6])), sparse_frac_k=float(rng.choice([0.0, 0.5, 1.0])),
                   sparse_frac_v=float(rng.choice([0.3, 1.0])), dense_first_tiles=int(rng.integers(0, 3)),
                   dense_last_tiles=int(rng.integers(0, 5)))
    else:
        sk, sv = _mixed_states(B, Hkv, T, seed=7000 + seed, p_skip=float(rng.choice([0.2, 0.8])))
        pol = dict(state_k=sk, state_v=sv)
    q = Q[:, :, 0, :].copy()
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, dtype=dtype, **pol)
    Or, Lr = orc.attention_decode(q, pk, pv)
    for ns in (1, int(rng.integers(2, 9))):
        O, LSE = hb.decode_attn(sh, _dev(q, dtype), kv, n_splits=ns)
        torch.cuda.synchronize()
        what = f"seed {seed}: B{B} Hq{Hq} Hkv{Hkv} T{T} {dtype} splits {ns} {sorted(pol)}"
        assert_close(_f32(O), Or, "decode " + what)
        assert_lse_close(LSE.cpu().numpy(), Lr, "decode lse " + what)


def test_explicit_states_on_the_device_run_with_no_host_wait():
    """A pruner that leaves its block-level masks on the device (Sec. III-A: the compressor takes the
    masks M as an input): compress with those states, causal prefill and decode are issued back to
    back on one stream with no host synchronisation in between (the states are produced by device
    work queued just before), and match the oracle."""
    B, Hq, Hkv, T = 2, 8, 2, 13
    L = 64 * T
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=300, k_outliers=True)
    sk, sv = _mixed_states(B, Hkv, T, seed=301, p_skip=0.2)
    sh = hb.make_shape(B, Hq, Hkv, L)
    Kd, Vd, Qd = _dev(K), _dev(V), _dev(Q)
    qd = _dev(Q[:, :, -1, :].copy())
    kv = hb.PackedKV(sh, [0, T, T, T, T])
    kv.uniform = 0
    stream = torch.cuda.Stream()
    stage = torch.from_numpy(np.stack([sk, sv])).cuda()          # uploaded before the stream work starts
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        # the "pruner": device work that produces the states on the same stream
        sk_d = (stage[0] + 0).contiguous()
        sv_d = (stage[1] + 0).contiguous()
        pol = hb.make_policy(state_k=sk_d, state_v=sv_d)
        hb.compress_kv(sh, pol, Kd, Vd, out=kv)
        O, LSE = hb.prefill_attn(sh, Qd, kv)
        Od, LSEd = hb.decode_attn(sh, qd, kv, n_splits=3)
    stream.synchronize()
    hb.check_state_flag(pol)
    pk, pv, _ = orc.compress_kv(K, V, state_k=sk, state_v=sv)
    check_packed_bit_exact(sh, kv, pk, pv)
    rows = wl.sample_rows(B, Hq, L, 150, seed=302, extra=[(0, 0, 0), (B - 1, Hq - 1, L - 1)])
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    assert_close(_f32(O)[idx], Or, "prefill after device-state compress")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "prefill after device-state compress lse")
    Odr, Ldr = orc.attention_decode(Q[:, :, -1, :].copy(), pk, pv)
    assert_close(_f32(Od), Odr, "decode after device-state compress")
    assert_lse_close(LSEd.cpu().numpy(), Ldr, "decode after device-state compress lse")


def test_explicit_states_into_pools_that_are_too_small():
    """Pools with fewer slots than the states ask for: the tiles that find no slot when their turn comes
    are left out of K and V, take no slot, and the flag goes up; the oracle walks the same counters."""
    B, Hq, Hkv, T = 2, 4, 2, 11
    L = 64 * T
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=310)
    sk, sv = _mixed_states(B, Hkv, T, seed=311, p_skip=0.1)
    caps = (2, 3, 3, 2)
    sh = hb.make_shape(B, Hq, Hkv, L)
    kv = hb.PackedKV(sh, [0, *caps])
    kv.uniform = 0
    pol = hb.make_policy(state_k=sk, state_v=sv)
    hb.compress_kv(sh, pol, _dev(K), _dev(V), out=kv)
    torch.cuda.synchronize()
    with pytest.raises(hb.HsError, match="more slots"):
        hb.check_state_flag(pol)
    pk, pv, info = orc.compress_kv(K, V, state_k=sk, state_v=sv, caps=caps)
    assert info["dropped"]
    check_packed_bit_exact(sh, kv, pk, pv)
    q = Q[:, :, 0, :].copy()
    O, LSE = hb.decode_attn(sh, _dev(q), kv, n_splits=2)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, pk, pv)
    assert_close(_f32(O), Or, "decode over capacity-limited pools")


def test_recompress_into_small_pools_then_append():
    """Further pruning into pools that are too small, then an append: the dropped tiles took no slot, so
    the appended tile gets a slot that no live tile uses (slots stay 0 .. n-1 per pool)."""
    B, Hq, Hkv, T = 2, 4, 2, 10
    L = 64 * T
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=320)
    # source: keys dense, values mixed; the last two tiles not filled yet
    sk = np.full((B, Hkv, T), orc.DENSE, dtype=np.int8)
    _, sv = _mixed_states(B, Hkv, T, seed=321, p_skip=0.0)
    sk[:, :, 8:], sv[:, :, 8:] = 0, 0
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, state_k=sk, state_v=sv)
    tk = np.full((B, Hkv, T), orc.SPARSE24, dtype=np.int8)
    tv = np.full((B, Hkv, T), orc.SPARSE24, dtype=np.int8)
    caps = (0, 5, 0, 7)                                      # 5 key slots for 8 tiles
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    kv2 = hb.recompress_kv(sh, kv, hb.make_policy(state_k=tk, state_v=tv), counts=[0, *caps], overflow=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1
    rk, rv, dropped = orc.recompress_kv(pk, pv, tk, tv, caps=caps)
    assert dropped
    check_packed_bit_exact(sh, kv2, rk, rv)
    assert (np.abs(rv.map).max(axis=-1) == 5).all()          # V holds 5 tiles too: the dropped ones took no V slot
    # append tile 8 as dense K? no dense pool: 2:4 K is full -> stays skipped, flag; V-only room does not help
    flag.zero_()
    Kd, Vd = _dev(K), _dev(V)
    hb.append_tile(sh, kv2, 8, Kd[:, :, 512:576].contiguous(), Vd[:, :, 512:576].contiguous(), overflow=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1 and (kv2.k_map[:, :, 8].cpu().numpy() == 0).all()
    # with room for one more key tile the append takes slot 5 (the 6th) in K and in V
    kv3 = hb.recompress_kv(sh, kv, hb.make_policy(state_k=tk, state_v=tv), counts=[0, 0, 6, 0, 7])
    rk3, rv3, _ = orc.recompress_kv(pk, pv, tk, tv, caps=(0, 6, 0, 7))
    # drop two tiles by hand so that room appears: recompress again towards a target that skips tiles 0, 1
    tk2, tv2 = tk.copy(), tv.copy()
    tk2[:, :, :2], tv2[:, :, :2] = 0, 0
    kv4 = hb.recompress_kv(sh, kv3, hb.make_policy(state_k=tk2, state_v=tv2), counts=[0, 0, 6, 0, 7])
    rk4, rv4, _ = orc.recompress_kv(rk3, rv3, tk2, tv2, caps=(0, 6, 0, 7))
    hb.append_tile(sh, kv4, 8, Kd[:, :, 512:576].contiguous(), Vd[:, :, 512:576].contiguous(), overflow=flag)
    orc.append_tile(rk4, rv4, 8, K[:, :, 512:576], V[:, :, 512:576], orc.SPARSE24, orc.SPARSE24)
    torch.cuda.synchronize()
    check_packed_bit_exact(sh, kv4, rk4, rv4)
    live = rk4.map[0, 0][rk4.map[0, 0] != 0]
    assert sorted((-live).tolist()) == list(range(1, live.size + 1))       # every slot used once
    q = Q[:, :, 0, :].copy()
    O, LSE = hb.decode_attn(sh, _dev(q), kv4, n_splits=2)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, rk4, rv4)
    assert_close(_f32(O), Or, "decode after recompress into small pools + append")


# ------------------------------------------------------------------ fp16 (the paper's element type)
# fp16 output rounding alone is 8x finer than bf16's, so the same bars leave more room; the values checked
# are the same ones as for bf16.
@pytest.mark.parametrize("pol", [dict(), dict(sparse_frac_k=0.0, sparse_frac_v=0.0), dict(sparse_frac_k=0.0),
                                 dict(skip_frac=0.25, sparse_frac_k=0.5, sparse_frac_v=0.7)])
def test_fp16_all_stages(pol):
    B, Hq, Hkv, L = 2, 8, 2, 64 * 12
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=180, k_outliers=True, dtype="fp16")
    K[0, 0, 5, :8] = wl.f32_to_f16_bits(np.array([1, 1, -1, 1, 0, -0.0, 0, 0], dtype=np.float32))    # ties and zeros
    V[0, 1, 8:12, 7] = wl.f32_to_f16_bits(np.array([6e-8, -6e-8, 1e-7, 0], dtype=np.float32))        # subnormals
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, dtype="fp16", **pol)
    check_packed_bit_exact(sh, kv, pk, pv)
    O, LSE = _prefill(sh, _dev(Q, "fp16"), kv)
    torch.cuda.synchronize()
    rows = wl.sample_rows(B, Hq, L, 160, seed=181, extra=[(0, 0, 0), (B - 1, Hq - 1, L - 1)])
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    assert_close(_f32(O)[idx], Or, f"fp16 prefill {sorted(pol)}")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "fp16 prefill lse")
    assert np.abs(_f32(O)[idx] - Or).mean() / np.abs(Or).mean() < 4e-4        # one fp16 term of P is enough
    q = Q[:, :, -1, :].copy()
    for ns in (0, 5):
        Od, LSEd = hb.decode_attn(sh, _dev(q, "fp16"), kv, n_splits=ns)
        torch.cuda.synchronize()
        Odr, Ldr = orc.attention_decode(q, pk, pv)
        assert_close(_f32(Od), Odr, f"fp16 decode {sorted(pol)} splits {ns}")
        assert_lse_close(LSEd.cpu().numpy(), Ldr, "fp16 decode lse")
    Kt, Vt = K[:, :, :64].copy(), V[:, :, :64].copy()
    Od, LSEd = hb.decode_attn(sh, _dev(q, "fp16"), kv, tail_k=_dev(Kt, "fp16"), tail_v=_dev(Vt, "fp16"), tail_len=9)
    torch.cuda.synchronize()
    Odr, Ldr = orc.attention_decode(q, pk, pv, tail_k=Kt, tail_v=Vt, tail_len=9)
    assert_close(_f32(Od), Odr, "fp16 decode with tail")


def test_fp16_large_logits_and_long_flat_rows():
    """fp16 numerators: the reference has to be renewed before a numerator reaches 65504 (keys that grow
    along the sequence), and small numerators of a long, flat row must not be flushed away."""
    B, Hq, Hkv, L = 1, 4, 1, 64 * 24
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=190, dtype="fp16")
    Kf = wl.f16_bits_to_f32(K)
    ramp = np.linspace(0.05, 6.0, L, dtype=np.float32)[None, None, :, None]     # logits grow to the hundreds
    Kb = wl.f32_to_f16_bits(Kf * ramp)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, Kb, V, dtype="fp16")
    O, LSE = _prefill(sh, _dev(Q, "fp16"), kv)
    Od, LSEd = hb.decode_attn(sh, _dev(Q[:, :, -1, :].copy(), "fp16"), kv)
    torch.cuda.synchronize()
    rows = [(0, h, i) for h in range(Hq) for i in range(0, L, 7)] + [(0, h, L - 1) for h in range(Hq)]
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    assert_close(_f32(O)[idx], Or, "fp16 prefill growing logits")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "fp16 prefill growing logits lse")
    Odr, Ldr = orc.attention_decode(Q[:, :, -1, :].copy(), pk, pv)
    assert_close(_f32(Od), Odr, "fp16 decode growing logits")
    # flat row: one key far above 1500 equal ones; the many small numerators carry weight together
    Kz = np.zeros_like(K)
    Kz[0, 0, 100] = wl.f32_to_f16_bits(Q[0, 0, -1].view(np.float16).astype(np.float32) * 1.23)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, Kz, V, dtype="fp16", sparse_frac_k=0.0, sparse_frac_v=0.0)
    Od, LSEd = hb.decode_attn(sh, _dev(Q[:, :, -1, :].copy(), "fp16"), kv, n_splits=1)
    O, LSE = _prefill(sh, _dev(Q, "fp16"), kv)
    torch.cuda.synchronize()
    Odr, Ldr = orc.attention_decode(Q[:, :, -1, :].copy(), pk, pv)
    assert_close(_f32(Od), Odr, "fp16 decode flat row")
    assert_lse_close(LSEd.cpu().numpy(), Ldr, "fp16 decode flat row lse")
    Or, Lr = orc.attention_rows(Q, pk, pv, [(0, 0, L - 1)], causal=True)
    assert_close(_f32(O)[0, 0, L - 1][None], Or, "fp16 prefill flat row")


# ------------------------------------------------------------------ edges and errors
@pytest.mark.parametrize("planted", ["tiny", "huge", "both"])
@pytest.mark.parametrize("pol", [dict(), dict(sparse_frac_k=0.0, sparse_frac_v=0.0), dict(sparse_frac_v=0.5),
                                 dict(skip_frac=0.25, sparse_frac_k=0.5, sparse_frac_v=0.7)])
def test_bf16_cache_with_both_v_tile_encodings(pol, planted):
    """V tiles of a bf16 cache whose stored values fp16 holds exactly carry the encoding bit and go
    through the fp16 matrix instructions; tiles with values under fp16's subnormal step or over its
    largest number stay bf16.  Both kinds in one row, in every kernel specialisation."""
    B, Hq, Hkv, L = 2, 8, 2, 64 * 14
    T = L // 64
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=190, k_outliers=True)
    Vf = wl.bf16_bits_to_f32(V)
    rng = np.random.default_rng(191)
    kind = rng.integers(0, 3, size=(B, Hkv, T))          # 0: as drawn, 1: tiny, 2: huge
    kind[0, 0, :] = 0                                       # one row with fp16 tiles only
    kind[1, 1, :] = 1 if planted != "huge" else 2           # one row with bf16 tiles only
    for b in range(B):
        for h in range(Hkv):
            for t in range(T):
                if kind[b, h, t] == 1 and planted in ("tiny", "both"):
                    Vf[b, h, 64 * t:64 * t + 64] *= 2.0 ** -20
                if kind[b, h, t] == 2 and planted in ("huge", "both"):
                    Vf[b, h, 64 * t:64 * t + 64] *= 2.0 ** 18
    V = wl.f32_to_bf16_bits(Vf)                             # exact: powers of two
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, **pol)
    flagged = pv.f16
    live = pv.map != 0
    assert (flagged & live).any() and (~flagged & live).any()
    check_packed_bit_exact(sh, kv, pk, pv)
    O, LSE = _prefill(sh, _dev(Q), kv)
    torch.cuda.synchronize()
    rows = wl.sample_rows(B, Hq, L, 200, seed=192, extra=[(0, 0, 0), (B - 1, Hq - 1, L - 1)])
    Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    got = _f32(O)[idx]
    if planted == "tiny":                                   # no huge tile hides the others' error
        assert_close(got, Or, f"prefill v encodings {sorted(pol)}")
    else:                                                   # per (b, h) row block: scales differ by 2^18
        for b in range(B):
            for h in range(Hq):
                sel = (idx[0] == b) & (idx[1] == h)
                if sel.any():
                    assert_close(got[sel], Or[sel], f"prefill v encodings {planted} b{b} h{h}")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "prefill v encodings lse")
    q = Q[:, :, -1, :].copy()
    Odr, Ldr = orc.attention_decode(q, pk, pv)
    for ns in (0, 3):
        Od, LSEd = hb.decode_attn(sh, _dev(q), kv, n_splits=ns)
        torch.cuda.synchronize()
        for b in range(B):
            for hk in range(Hkv):
                g = slice(hk * (Hq // Hkv), (hk + 1) * (Hq // Hkv))
                assert_close(_f32(Od)[b, g], Odr[b, g], f"decode v encodings {planted} splits {ns} b{b} hkv{hk}")
        assert_lse_close(LSEd.cpu().numpy(), Ldr, "decode v encodings lse")


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_recompress_explicit_states_bit_exact_and_attention(dtype):
    """Further pruning of a packed cache (dense -> 2:4, anything -> dropped, the rest carried over) against
    the oracle, bit for bit, then attention over the result."""
    B, Hq, Hkv, L = 2, 8, 2, 64 * 19
    T = L // 64
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=210, k_outliers=True, dtype=dtype)
    if dtype == "bf16":
        Vf = wl.bf16_bits_to_f32(V)
        Vf[:, :, 64 * 2:64 * 3:4] = 2.0 ** -40          # dense form not exact in fp16, 2:4 form exact
        Vf[:, :, 64 * 3:64 * 4] *= 2.0 ** -22           # never exact
        V = wl.f32_to_bf16_bits(Vf)
    sk, sv = _mixed_states(B, Hkv, T, seed=211, p_skip=0.15)
    sk[:, :, 2:4], sv[:, :, 2:4] = 1, 1
    tk, tv = _mixed_states(B, Hkv, T, seed=212, p_skip=0.15)
    tk[:, :, 2:4], tv[:, :, 2:4] = 2, 2
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, dtype=dtype, state_k=sk, state_v=sv)
    kv2 = hb.recompress_kv(sh, kv, hb.make_policy(state_k=tk, state_v=tv))
    torch.cuda.synchronize()
    rk, rv = orc.recompress_kv(pk, pv, tk, tv)
    check_packed_bit_exact(sh, kv2, rk, rv)
    check_packed_bit_exact(sh, kv, pk, pv)                  # the source is untouched
    O, LSE = hb.prefill_attn(sh, _dev(Q, dtype), kv2)
    torch.cuda.synchronize()
    rows = wl.sample_rows(B, Hq, L, 120, seed=213, extra=[(B - 1, Hq - 1, L - 1)])
    Or, Lr = orc.attention_rows(Q, rk, rv, rows, causal=True)
    idx = tuple(np.array(rows).T)
    assert_close(_f32(O)[idx], Or, f"prefill after recompress {dtype}")
    assert_lse_close(LSE.cpu().numpy()[idx], Lr, "prefill after recompress lse")
    q = Q[:, :, -1, :].copy()
    Od, LSEd = hb.decode_attn(sh, _dev(q, dtype), kv2, n_splits=3)
    torch.cuda.synchronize()
    Odr, Ldr = orc.attention_decode(q, rk, rv)
    assert_close(_f32(Od), Odr, f"decode after recompress {dtype}")
    assert_lse_close(LSEd.cpu().numpy(), Ldr, "decode after recompress lse")


@pytest.mark.parametrize("first,last", [(0, 0), (1, 3)])
def test_recompress_prefill_policy_to_decode_policy(first, last):
    """The paper's differentiated setting: prefill with keys dense and values 2:4, then every key tile
    pruned for decode (optionally sink / local-window tiles kept dense).  Equals compressing the
    original tensors with the decode policy, on the GPU and in the oracle."""
    B, Hq, Hkv, L = 1, 8, 2, 64 * 16
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=220, k_outliers=True)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, sparse_frac_k=0.0, sparse_frac_v=1.0)
    assert kv.uniform == 1
    tgt = dict(sparse_frac_k=1.0, sparse_frac_v=1.0, dense_first_tiles=first, dense_last_tiles=last)
    kv2 = hb.recompress_kv(sh, kv, hb.make_policy(**tgt))
    torch.cuda.synchronize()
    assert kv2.uniform == (1 if first + last == 0 else 0)
    sh2, kv_direct, ck, cv, info = compress_both(B, Hq, Hkv, L, K, V, **tgt)
    rk, rv = orc.recompress_kv(pk, pv, info["state_k"], info["state_v"])
    check_packed_bit_exact(sh, kv2, rk, rv)
    # V was 2:4 everywhere already: its protected tiles cannot go back to dense; K equals the direct result
    assert (rv.map < 0).all() and (rk.map == ck.map).all()
    Ku, _ = hb.unpack_kv(sh, kv2)
    Kd, _ = hb.unpack_kv(sh, kv_direct)
    torch.cuda.synchronize()
    assert torch.equal(Ku.view(torch.int16), Kd.view(torch.int16))
    q = Q[:, :, 0, :].copy()
    Od, LSEd = hb.decode_attn(sh, _dev(q), kv2)
    torch.cuda.synchronize()
    Odr, Ldr = orc.attention_decode(q, rk, rv)
    assert_close(_f32(Od), Odr, "decode after recompress to S_K=1")
    assert_lse_close(LSEd.cpu().numpy(), Ldr, "decode after recompress lse")


def test_recompress_ranked_targets_from_kept_tile_scores():
    """Decode-phase policy with fractions (skip the quietest quarter, half of the key tiles 2:4 by lowest
    pruning loss, sink and local-window tiles dense) applied to a prefill cache (keys dense, values 2:4): the
    ranking uses the tile scores taken from the original tensors (hs_score_tiles), which equal the oracle's,
    and the result equals the oracle's further pruning towards the states that policy gives the originals."""
    B, Hq, Hkv, T = 2, 8, 2, 24
    L = 64 * T
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=330, k_outliers=True)
    K[0, 0, 64 * 9:64 * 10] = K[0, 0, 64 * 3:64 * 4]           # an exact tie in energy and in loss
    V[0, 0, 64 * 9:64 * 10] = V[0, 0, 64 * 3:64 * 4]
    Kd, Vd = _dev(K), _dev(V)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, sparse_frac_k=0.0, sparse_frac_v=1.0)
    scores = hb.score_tiles(sh, Kd, Vd)
    tgt = dict(skip_frac=0.25, sparse_frac_k=0.5, sparse_frac_v=1.0, dense_first_tiles=1, dense_last_tiles=2)
    _, _, info = orc.compress_kv(K, V, **tgt)                    # states the policy gives the original tensors
    torch.cuda.synchronize()
    sc = scores.cpu().numpy()
    for plane, key in enumerate(("energy", "loss_k", "loss_v")):
        assert np.allclose(sc[plane], info[key], rtol=1e-12, atol=0.0), key
        srt = np.sort(info[key], axis=-1)
        gaps = np.diff(srt, axis=-1) / srt[..., 1:]
        assert ((gaps > 1e-12) | (gaps == 0)).all()              # no cut on a rounding-level near-tie
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    kv2 = hb.recompress_kv(sh, kv, hb.make_policy(tile_scores=scores, **tgt), overflow=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0 and kv2.uniform == 0
    rk, rv = orc.recompress_kv(pk, pv, info["state_k"], info["state_v"])
    check_packed_bit_exact(sh, kv2, rk, rv)
    assert int((rk.map == 0).sum()) == B * Hkv * 5 and (rv.map[:, :, 0] < 0).all()      # V was 2:4 already: stays
    q = Q[:, :, 0, :].copy()
    O, LSE = hb.decode_attn(sh, _dev(q), kv2, n_splits=3)
    torch.cuda.synchronize()
    Or, Lr = orc.attention_decode(q, rk, rv)
    assert_close(_f32(O), Or, "decode after ranked recompress")
    assert_lse_close(LSE.cpu().numpy(), Lr, "decode after ranked recompress lse")


@pytest.mark.parametrize("T,first,last", [(1, 0, 0), (3, 1, 1), (64, 0, 0), (65, 0, 0), (130, 1, 4), (257, 0, 0), (1024, 2, 3), (2048, 0, 0), (2049, 1, 0)])
def test_selection_of_given_scores(T, first, last):
    """The n lowest (score, tile index), for scores of every kind: all equal, more and fewer equal ones than one wave
    ranks at once, differing only in the lowest or only in the highest bits, zeros, infinities."""
    rng = np.random.default_rng(T)
    kinds = [np.full(T, 3.25), rng.integers(0, 2, T) * 1.0, rng.integers(0, 7, T) * 0.5, 1.0 + rng.integers(0, 9, T) * 2.0 ** -52,
             rng.random(T), 10.0 ** rng.uniform(-300, 300, T), 8192 + rng.standard_normal(T), np.where(rng.random(T) < 0.4, np.inf, rng.random(T))]
    Hkv = len(kinds)
    sh = hb.make_shape(1, Hkv, Hkv, 64 * T)
    scores = np.stack([np.stack(kinds), np.stack(kinds[1:] + kinds[:1]), np.stack(kinds[3:] + kinds[:3])])[:, None]
    x = torch.ones(1, Hkv, 64 * T, 128, device="cuda", dtype=torch.bfloat16)
    kv = hb.compress_kv(sh, hb.make_policy(sparse_frac_k=0.0, sparse_frac_v=0.0), x, x)
    del x
    for skip, fk, fv in ((0.25, 0.5, 0.3), (0.5, 1.0, 0.99), (0.0, 0.01, 1.0), (0.97, 0.5, 0.5)):
        pol = hb.make_policy(skip_frac=skip, sparse_frac_k=fk, sparse_frac_v=fv, dense_first_tiles=first, dense_last_tiles=last,
                             tile_scores=torch.from_numpy(scores).cuda())
        out = hb.recompress_kv(sh, kv, pol, counts=[0, T, T, T, T])
        km, vm = lib_maps(out.k_map, out.v_map)[:2]
        for h in range(Hkv):
            mid = np.arange(first, T - last)
            order = mid[np.lexsort((mid, scores[0, 0, h, mid]))]
            n_skip = int(np.floor(skip * len(mid)))
            kept = np.sort(order[n_skip:])
            want = np.ones((2, T), dtype=np.int64)
            want[:, order[:n_skip]] = 0
            for x_, f in ((0, fk), (1, fv)):
                want[x_, kept[np.lexsort((kept, scores[1 + x_, 0, h, kept]))][:int(np.floor(f * len(kept)))]] = -1
            assert (np.sign(np.asarray(km)[0, h]) == want[0]).all() and (np.sign(np.asarray(vm)[0, h]) == want[1]).all(), (h, skip, fk, fv)


@pytest.mark.parametrize("Hkv,T", [(2, 1), (2, 40), (3, 257), (8, 600)])                 # one launch; (8, 600): two
@pytest.mark.parametrize("room", [1.0, 0.6])
def test_recompress_maps_are_those_of_a_walk_in_tile_order(Hkv, T, room):
    """Slots of the new cache, the encoding bit of tiles that keep their kind, tiles left out where a pool is full,
    and both bits of the flag, for explicit targets with invalid pairs among them."""
    rng = np.random.default_rng(T)
    sk, sv = _mixed_states(1, Hkv, T, seed=T, p_skip=0.2)
    sh = hb.make_shape(1, Hkv, Hkv, 64 * T)
    g = torch.Generator(device="cuda").manual_seed(T)
    K, V = (torch.randn((1, Hkv, 64 * T, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    kv = hb.compress_kv(sh, hb.make_policy(state_k=sk, state_v=sv), K, V)
    tk, tv = rng.integers(0, 3, (1, Hkv, T)).astype(np.int8), rng.integers(0, 3, (1, Hkv, T)).astype(np.int8)
    tgt = hb.make_policy(state_k=torch.from_numpy(tk).cuda(), state_v=torch.from_numpy(tv).cuda())
    rank = {1: 0, 2: 1, 0: 2}
    new = np.zeros((2, Hkv, T), dtype=np.int64)
    invalid = False
    for h in range(Hkv):
        for t in range(T):
            a, b = int(tk[0, h, t]), int(tv[0, h, t])
            if (a == 0) != (b == 0):
                invalid, a, b = True, 1, 1
            n = [max((int(s), x), key=lambda v: rank[v]) for s, x in ((sk[0, h, t], a), (sv[0, h, t], b))]
            new[:, h, t] = 0 if 0 in n else n
    caps = [0] + [max(1, int(np.ceil(room * (new[x] == k).sum(-1).max()))) for x, k in ((0, 1), (0, 2), (1, 1), (1, 2))]
    over = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = hb.recompress_kv(sh, kv, tgt, counts=caps, overflow=over)
    km, vm, f16 = lib_maps(out.k_map, out.v_map)
    old = lib_maps(kv.k_map, kv.v_map)
    full = False
    for h in range(Hkv):
        c = {(x, k): 0 for x in (0, 1) for k in (1, 2)}
        for t in range(T):
            a, b = new[:, h, t]
            want = (0, 0)
            if a:
                if c[0, a] < caps[a] and c[1, b] < caps[2 + b]:
                    c[0, a] += 1
                    c[1, b] += 1
                    want = (c[0, a] * (1 if a == 1 else -1), c[1, b] * (1 if b == 1 else -1))
                else:
                    full = True
            assert (km[0, h, t], vm[0, h, t]) == want, (h, t)
            if want[1] and (want[1] > 0) == (old[1][0, h, t] > 0):
                assert f16[0, h, t] == old[2][0, h, t]
    assert int(over.item()) == int(full) + 2 * int(invalid)


def test_recompress_capacity_overflow_and_argument_errors():
    B, Hq, Hkv, L = 1, 4, 1, 64 * 8
    T = L // 64
    _, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, 1, seed=230)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V, sparse_frac_k=0.0, sparse_frac_v=0.0)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    # room for 5 of the 8 key tiles: the first 5 tiles survive, the rest is left out of K and V alike
    kv2 = hb.recompress_kv(sh, kv, hb.make_policy(), counts=[0, 0, 5, 0, T], overflow=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1
    assert kv2.k_map.cpu().numpy().reshape(-1).tolist() == [-1, -2, -3, -4, -5, 0, 0, 0]
    vm = kv2.v_map.cpu().numpy().reshape(-1)
    assert ((np.abs(vm) & ~hb.MAP_F16) == [1, 2, 3, 4, 5, 0, 0, 0]).all() and (vm <= 0).all()
    flag.zero_()
    hb.recompress_kv(sh, kv, hb.make_policy(), overflow=flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    with pytest.raises(hb.HsError):                         # a ranked target needs the tile scores
        hb.recompress_kv(sh, kv, hb.make_policy(sparse_frac_k=0.5))
    with pytest.raises(hb.HsError):
        hb.recompress_kv(sh, kv, hb.make_policy(skip_frac=0.25))
    import ctypes as C
    a = kv.struct()
    ws = torch.empty(hb.workspace_bytes(sh, 3), dtype=torch.uint8, device="cuda")
    pol = hb.make_policy()
    assert hb.lib().hs_recompress_kv(C.byref(sh), C.byref(pol), C.byref(a), C.byref(a), ws.data_ptr(), None, None) == -1


def test_single_tile_and_odd_batch_shapes():
    """L = 64 (one tile, one split), B = 3, 3 KV heads: smallest grid dimensions on every kernel."""
    for (B, Hq, Hkv, L) in ((1, 1, 1, 64), (3, 6, 3, 64 * 3), (2, 16, 2, 64 * 2)):
        Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=130 + B)
        sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, K, V)
        check_packed_bit_exact(sh, kv, pk, pv)
        O, LSE = _prefill(sh, _dev(Q), kv)
        q = Q[:, :, -1, :].copy()
        Od, LSEd = hb.decode_attn(sh, _dev(q), kv)
        torch.cuda.synchronize()
        rows = [(b, h, i) for b in range(B) for h in range(Hq) for i in range(L)]
        Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True)
        assert_close(_f32(O).reshape(-1, 128), Or, f"prefill B{B} Hq{Hq} Hkv{Hkv} L{L}")
        Odr, Ldr = orc.attention_decode(q, pk, pv)
        assert_close(_f32(Od), Odr, f"decode B{B} Hq{Hq} Hkv{Hkv} L{L}")
        assert_lse_close(LSEd.cpu().numpy(), Ldr, "decode lse")


def test_scale_argument_and_large_logits():
    """Explicit softmax scale, and keys scaled so that logits reach the hundreds (the lazily
    updated softmax reference must follow without overflow)."""
    B, Hq, Hkv, L = 1, 4, 1, 64 * 6
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=140)
    Kbig = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(K) * 24.0)
    # a late tile with much larger keys: the reference has to jump upwards mid-sequence
    Kbig[:, :, 64 * 4:64 * 5] = wl.f32_to_bf16_bits(wl.bf16_bits_to_f32(K[:, :, 64 * 4:64 * 5]) * 96.0)
    sh, kv, pk, pv, _ = compress_both(B, Hq, Hkv, L, Kbig, V)
    for scale in (0.0, 0.25):
        O, LSE = _prefill(sh, _dev(Q), kv, scale=scale)
        Od, LSEd = hb.decode_attn(sh, _dev(Q[:, :, -1, :].copy()), kv, scale=scale)
        torch.cuda.synchronize()
        rows = [(0, h, i) for h in range(Hq) for i in range(L)]
        Or, Lr = orc.attention_rows(Q, pk, pv, rows, causal=True, scale=None if scale == 0.0 else scale)
        assert_close(_f32(O).reshape(-1, 128), Or, f"prefill large logits scale={scale}")
        assert_lse_close(LSE.cpu().numpy().reshape(-1), Lr, f"prefill large logits lse scale={scale}")
        Odr, Ldr = orc.attention_decode(Q[:, :, -1, :].copy(), pk, pv, scale=None if scale == 0.0 else scale)
        assert_close(_f32(Od), Odr, f"decode large logits scale={scale}")


def test_matrix_rate_probe_runs_and_counts_its_work():
    """The benchmark's register-resident matrix-instruction loop: runs, reports the flops of the launch
    (2 workgroups per compute unit x 4 waves x 8 instructions x iterations x 2*16*16*K) and the clocks spent."""
    import ctypes as C
    sink = torch.zeros(4, dtype=torch.int64, device="cuda")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for kind, k in ((0, 32), (1, 64)):
        flop = hb.probe_mfma_rate(kind, 500, sink)
        torch.cuda.synchronize()
        assert flop == 2 * cus * 4 * 8 * 500 * 2 * 16 * 16 * k
        clocks, ticks, _, never = sink.cpu().tolist()
        assert clocks > 500 * 8 * 8 and ticks > 0 and never == 0     # >= 8 clocks per matrix instruction
    f = C.c_double(0.0)
    assert hb.lib().hs_probe_mfma_rate(2, 10, sink.data_ptr(), C.byref(f), None) == -1
    assert hb.lib().hs_probe_mfma_rate(0, 0, sink.data_ptr(), C.byref(f), None) == -1


def test_stream_read_probe_runs():
    """The benchmark's load-only kernel (the decode kernel's access pattern): runs over a buffer of pool-shaped
    regions, with and without its epilogue, and rejects shapes it cannot split evenly."""
    n_tiles, n_wg = 512, 32
    buf = torch.ones(n_tiles * 18432, dtype=torch.uint8, device="cuda")
    sink = torch.zeros(16 + 512 * n_wg, dtype=torch.float32, device="cuda")
    hb.probe_stream_read(buf, n_tiles, n_wg, True, sink)
    torch.cuda.synchronize()
    # every byte is 1: each lane's xor over 4 x 18 tiles' words ends up 0 -> the combined partials are 0
    assert float(sink[16:].abs().max().item()) == 0.0
    hb.probe_stream_read(buf, n_tiles, n_wg, False, sink)
    torch.cuda.synchronize()
    with pytest.raises(hb.HsError):
        hb.probe_stream_read(buf, n_tiles, 24, True, sink)            # 512 tiles do not split over 24 workgroups of 4 waves


def test_argument_errors_on_device_calls():
    B, Hq, Hkv, L = 1, 4, 1, 256
    Q, K, V = wl.make_qkv(B, Hq, Hkv, L, 128, L, seed=150)
    sh = hb.make_shape(B, Hq, Hkv, L)
    Kd, Vd = _dev(K), _dev(V)
    # pools sized for an all-2:4 policy cannot take a policy that needs dense tiles
    kv = hb.PackedKV(sh, hb.tile_counts(sh, hb.make_policy()))
    with pytest.raises(hb.HsError):
        hb.compress_kv(sh, hb.make_policy(sparse_frac_k=0.5), Kd, Vd, out=kv)
    # explicit states: a tile skipped in K only is inconsistent.  Host arrays are checked by the binding;
    # states that are already on the device are checked by the kernel that turns them into maps: the tile
    # is stored as SKIP and bit 1 of the policy's flag goes up
    sk = np.array([[[2, 0, 2, 2]]], dtype=np.int8)
    sv = np.array([[[2, 2, 2, 7]]], dtype=np.int8)
    with pytest.raises(hb.HsError):
        hb.make_policy(state_k=sk, state_v=sv)
    pol_dev = hb.make_policy(state_k=torch.from_numpy(sk).cuda(), state_v=torch.from_numpy(sv).cuda())
    kv.uniform = 0
    hb.compress_kv(sh, pol_dev, Kd, Vd, out=kv)
    torch.cuda.synchronize()
    assert kv.k_map.cpu().numpy().reshape(-1).tolist() == [-1, 0, -2, 0]
    assert (np.abs(kv.v_map.cpu().numpy().reshape(-1)) & ~hb.MAP_F16).tolist() == [1, 0, 2, 0]
    with pytest.raises(hb.HsError, match="not valid"):
        hb.check_state_flag(pol_dev)
    kv = hb.compress_kv(sh, hb.make_policy(), Kd, Vd)
    # Lq not a multiple of the tile, Lq > L
    import ctypes as C
    kvs = kv.struct()
    Qd = _dev(Q)
    O = torch.empty_like(Qd)
    one = sh.B * sh.Hq * 64 * 129 * 4
    ws = torch.empty(2 * one, dtype=torch.uint8, device="cuda")
    for slab, n, w, room in ((8, 1, ws, 2 * one), (48, 1, ws, 2 * one), (32, 0, ws, 2 * one), (16, 65536, ws, 2 * one), (16, 3, ws, 2 * one),
                             (32, 2, ws, 2 * one - 1), (32, 2, None, 2 * one)):      # no such slab, no such ranges, no room for them
        assert hb.lib().hs_prefill_attn_planned(C.byref(sh), 64, 0, 0.0, 1, hb._ptr(Qd), C.byref(kvs), hb._ptr(O), None, hb._ptr(w), room, slab, n,
                                                None) == -1
    assert hb.lib().hs_prefill_attn(C.byref(sh), 100, 0.0, 1, hb._ptr(Qd), C.byref(kvs), hb._ptr(O), None, None, None) == -2
    assert hb.lib().hs_prefill_attn(C.byref(sh), 512, 0.0, 1, hb._ptr(Qd), C.byref(kvs), hb._ptr(O), None, None, None) == -1
    # a pool of more than 4 GiB per (batch, kv head) row: prefill addresses tiles with 32-bit offsets
    kvs.cap_sparse_v = (1 << 32) // 8192 + 1
    assert hb.lib().hs_prefill_attn(C.byref(sh), 256, 0.0, 1, hb._ptr(Qd), C.byref(kvs), hb._ptr(O), None, None, None) == -2
    kvs = kv.struct()
    # a uniform promise that the capacities contradict
    kvs.cap_sparse_k = 2
    assert hb.lib().hs_decode_attn(C.byref(sh), 0.0, 0, hb._ptr(Qd), C.byref(kvs), hb._ptr(O), None, hb._ptr(O), None) == -1
    torch.cuda.synchronize()
