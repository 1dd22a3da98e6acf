"""The work a user of this framework has it do, as cases that can be timed and checked.

A case is one call of the public entry points (paper_2604_16864_amd.binding) on a Llama-3.1-8B-like attention geometry or a
generic one: compress a K/V cache, append a full tile to a growing cache, prune a prefill cache further for decode, prefill
attention (whole prompt, chunk, short turn on a long context) and decode attention (single sequence, batch, serving step with
sequences of different length and a dense tail).  `prepare` makes inputs and the packed cache from a seed on the GPU, `run`
is the call, `exact` the same result from plain torch in 64 bits.

Fields of a case: op; B, Hq, Hkv, L (tokens the cache can hold), dtype; the pruning policy (skip, sk, sv, first, last: see
hs_policy); outliers (per-channel key scales log-uniform in [0.1, 10]); used = share of L the longest row holds (1: all of it);
ragged (rows hold different numbers of tiles); Lq (prefill queries, at the end of what the cache holds); tail (dense tail of
decode: "none", "one" length, "rows" lengths); entry (decode: "plain" allocates per call, "kept" passes buffers the program
keeps, "static" uses the library's own scratch); n_new (append: tiles per call, 0 = one tile per batch row at its own place).
"""
import math

import torch

from paper_2604_16864_amd import binding as hb

D, TILE = 128, 64

_BASE = dict(B=1, Hq=32, Hkv=8, L=32768, dtype="bf16", skip=0.0, sk=1.0, sv=1.0, first=0, last=0, outliers=False,
             used=1.0, ragged=False)


def _case(name, op, **kw):
    return dict(_BASE, name=name, op=op, **kw)


def listed():
    return [
        # the smallest call of all: one token of one GQA group over a 2K context
        _case("decode_2k", "decode", B=1, Hq=4, Hkv=1, L=2048, tail="none", entry="plain"),
        # one token of an 8B-class model over a 32K context, keys with outlier channels (the benchmark's decode)
        _case("decode_32k", "decode", outliers=True, tail="none", entry="kept"),
        # the largest: batch 8 at 128K with half of the tiles dropped
        _case("decode_b8_128k_skip50", "decode", B=8, L=131072, skip=0.5, tail="none", entry="kept"),
        # a serving step: 16 sequences of different length in one cache, sink and local window kept dense, and the
        # tokens of the tile not yet full in the dense tail
        _case("decode_serving_b16", "decode", B=16, L=16384, first=1, last=4, ragged=True, tail="rows", entry="kept"),
        # half of the key blocks pruned, all value blocks: the paper's intermediate setting, in its element type
        _case("decode_b4_32k_half_keys", "decode", B=4, dtype="fp16", sk=0.5, tail="one", entry="plain"),
        # prompt of 16K tokens
        _case("prefill_16k", "prefill", L=16384, Lq=16384),
        # prompt of 64K tokens at the highest hierarchical sparsity
        _case("prefill_64k_skip75", "prefill", L=65536, Lq=65536, skip=0.75),
        # one 2K chunk of a chunked prefill, 12K tokens already there, in a cache allocated for 32K; dense keys and
        # 2:4 values (the paper's quality-preserving setting)
        _case("prefill_chunk_2k", "prefill", dtype="fp16", sk=0.0, Lq=2048, used=0.4375),
        # a follow-up turn of 64 tokens on a 32K context
        _case("prefill_turn_64", "prefill", outliers=True, Lq=64),
        # compression with ranking: a quarter of the tiles dropped, half of the keys 2:4, sink and window dense
        _case("compress_ranked_32k", "compress", skip=0.25, sk=0.5, first=1, last=4, outliers=True),
        # every 64 steps of serving: the full tail tile of 16 sequences goes into the packed cache
        _case("append_b16", "append", B=16, L=8192, first=1, last=4, ragged=True, n_new=0),
        # after prefill with dense keys the cache is pruned further for decode
        _case("recompress_32k", "recompress", sk=0.0, first=1, last=4, outliers=True),
    ]


# ------------------------------------------------------------------------------------------------------------------
# draw
# ------------------------------------------------------------------------------------------------------------------
_POLICIES = [dict(), dict(), dict(sk=0.0), dict(sk=0.0, sv=0.0), dict(sk=0.5), dict(sk=0.5, sv=0.5), dict(skip=0.25),
             dict(skip=0.5), dict(skip=0.75), dict(first=1, last=4), dict(skip=0.5, sk=0.5, sv=0.75, first=1, last=4)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode"] * 4 + ["prefill"] * 3 + ["compress", "append", "recompress"])
    c = dict(_BASE, op=op, dtype=rng.choice(["bf16", "bf16", "fp16"]), outliers=rng.random() < 0.3)
    c["Hkv"] = rng.choice([1, 2, 3, 4, 8, 8, 8])
    c["Hq"] = c["Hkv"] * rng.choice([1, 2, 3, 4, 4, 4, 5, 7, 8])
    c["B"] = rng.choice([1, 1, 1, 2, 3, 4, 8, 13, 16])
    c.update(rng.choice(_POLICIES))
    rows = c["B"] * c["Hkv"]
    if op == "decode":
        T = _log_int(rng, 1, min(2048, 65536 // rows))      # at most half of the largest listed cache
        c["tail"] = rng.choice(["none", "one", "rows"])
        c["entry"] = rng.choice(["plain", "kept", "static"]) if c["tail"] == "none" else rng.choice(["plain", "kept"])
        c["ragged"] = c["tail"] == "rows" and c["B"] > 1
    elif op == "prefill":
        T = _log_int(rng, 1, 1024)
        Tq = _log_int(rng, 1, T)
        while c["B"] * c["Hq"] * Tq * (T - Tq / 2) * 4096 > 1.0e10:   # (query, token) pairs
            if c["B"] > 1:
                c["B"] -= 1
            elif Tq > 1:
                Tq //= 2
            else:
                T //= 2
        c["Lq"] = Tq * TILE
    elif op == "append":
        T = _log_int(rng, 2, min(2048, 65536 // rows))
        c["n_new"] = rng.choice([0, 1, 1, min(T - 1, rng.choice([2, 3, 8, 32, 64]))])
        c["ragged"] = c["n_new"] == 0 and c["B"] > 1
        c["used"] = 0.9
    else:
        T = _log_int(rng, 4, min(2048, 32768 // rows))
        if op == "recompress":                               # a prefill cache that decode prunes to 2:4 in both tensors
            c.update(skip=0.0, sk=0.0, sv=rng.choice([0.0, 1.0]), first=rng.choice([0, 1]), last=rng.choice([0, 4]))
    if c["ragged"]:                                          # explicit states: fractions other than 0 and 1 do not apply
        c.update(skip=0.0, sk=float(c["sk"] >= 0.5), sv=float(c["sv"] >= 0.5))
    c["L"] = T * TILE
    return c


# ------------------------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------------------------
def _dtype(c):
    return torch.float16 if c["dtype"] == "fp16" else torch.bfloat16


def _gen(seed, k):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 16 + k)


def _normal(shape, dtype, g):
    return torch.randn(shape, dtype=torch.float32, device="cuda", generator=g).to(dtype)


def _kv_tensor(c, seed, k, tokens, scaled):
    """[B, Hkv, tokens, D], drawn one batch row at a time (bounds the fp32 intermediate)."""
    g = _gen(seed, k)
    scale = None
    if scaled:
        u = torch.rand((c["Hkv"], 1, D), device="cuda", generator=_gen(seed, 7))
        scale = torch.exp(math.log(0.1) + u * math.log(100.0))
    out = torch.empty((c["B"], c["Hkv"], tokens, D), dtype=_dtype(c), device="cuda")
    for b in range(c["B"]):
        x = torch.randn(out.shape[1:], dtype=torch.float32, device="cuda", generator=g)
        out[b] = (x * scale if scale is not None else x).to(out.dtype)
    return out


def _held_tiles(c, seed):
    """Tiles each batch row holds: all of the capacity, a share of it, or (ragged) different shares."""
    T = c["L"] // TILE
    top = max(1, int(T * c["used"]))
    if c["op"] == "append":
        top = min(top, T - max(1, c["n_new"]))
    if not c["ragged"]:
        return [top] * c["B"]
    u = torch.rand(c["B"], generator=torch.Generator().manual_seed(int(seed) * 16 + 5)).tolist()
    return [max(1, min(top, int(round(top * (0.25 + 0.75 * x))))) for x in u]


def _explicit(c):
    return c["ragged"] or c["used"] < 1.0 or c["op"] == "append"


def _held_states(c, held):
    """Tile states of a cache that holds `held` tiles per row: sink and window dense, the middle 2:4 or dense, the rest SKIP."""
    T = c["L"] // TILE
    sk = torch.zeros((c["B"], c["Hkv"], T), dtype=torch.int8)
    sv = torch.zeros_like(sk)
    for b, n in enumerate(held):
        sk[b, :, :n] = hb.SPARSE24 if c["sk"] >= 0.5 else hb.DENSE
        sv[b, :, :n] = hb.SPARSE24 if c["sv"] >= 0.5 else hb.DENSE
        for s in (sk, sv):
            s[b, :, :min(c["first"], n)] = hb.DENSE
            s[b, :, max(0, n - c["last"]):n] = hb.DENSE
    return sk, sv


def _zeroed(shape, counts):
    kv = hb.PackedKV(shape, counts, "cuda")
    for t in (kv.k_dense, kv.k_nnz, kv.k_meta, kv.v_dense, kv.v_nnz, kv.v_meta, kv.k_map, kv.v_map):
        if t is not None:
            t.zero_()
    return kv


def _policy(c):
    return hb.make_policy(skip_frac=c["skip"], sparse_frac_k=c["sk"], sparse_frac_v=c["sv"], dense_first_tiles=c["first"],
                          dense_last_tiles=c["last"])


def _packed(c, seed, shape, K, V):
    """The packed cache a program holds before the call."""
    if not _explicit(c):
        return hb.compress_kv(shape, _policy(c), K, V)
    held = _held_tiles(c, seed)
    sk, sv = _held_states(c, held)
    pol = hb.make_policy(state_k=sk.numpy(), state_v=sv.numpy())
    # capacities a program allocates ahead: the protected tiles dense, the middle 2:4 (or all dense), tiles that come 2:4
    T, prot, n = c["L"] // TILE, min(c["L"] // TILE, c["first"] + c["last"]), max(1, c["n_new"]) if c["op"] == "append" else 0
    counts = [0]
    for f in (c["sk"], c["sv"]):
        counts += [prot, T] if f >= 0.5 else [T, n]
    kv = hb.compress_kv(shape, pol, K, V, out=_zeroed(shape, counts))
    hb.check_state_flag(pol)
    return kv


def _tail(c, seed):
    """Dense tail tensors and lengths (1..63 tokens generated since the last full tile)."""
    tk, tv = _kv_tensor(c, seed, 3, TILE, c["outliers"]), _kv_tensor(c, seed, 4, TILE, False)
    g = torch.Generator().manual_seed(int(seed) * 16 + 6)
    lens = torch.randint(1, TILE, (c["B"],), generator=g, dtype=torch.int32)
    return tk, tv, lens if c["tail"] == "rows" else lens[:1].expand(c["B"]).contiguous()


def prepare(case, seed):
    c = dict(case)
    shape = hb.make_shape(c["B"], c["Hq"], c["Hkv"], c["L"], dtype=_dtype(c))
    st = {"case": c, "shape": shape}
    K, V = _kv_tensor(c, seed, 1, c["L"], c["outliers"]), _kv_tensor(c, seed, 2, c["L"], False)
    if c["op"] == "compress":
        st.update(K=K, V=V, policy=_policy(c))
        return st
    st["kv"] = _packed(c, seed, shape, K, V)
    if c["op"] == "append":
        n = max(1, c["n_new"])
        st["K_new"], st["V_new"] = _kv_tensor(c, seed, 3, TILE * n, c["outliers"]), _kv_tensor(c, seed, 4, TILE * n, False)
        held = _held_tiles(c, seed)
        st["at"] = held[0] if c["n_new"] else torch.tensor(held, dtype=torch.int32, device="cuda")
    elif c["op"] == "recompress":
        st["target"] = hb.make_policy(dense_first_tiles=c["first"], dense_last_tiles=c["last"])
        st["counts"] = hb.tile_counts(shape, st["target"])
        if c["sv"] == 1.0:                                   # values are 2:4 already: their pools keep their sizes
            st["counts"][3:] = st["kv"].counts[3:]
    elif c["op"] == "prefill":
        st["Q"] = _normal((c["B"], c["Hq"], c["Lq"], D), _dtype(c), _gen(seed, 0))
        st["q_start"] = None if c["used"] == 1.0 else _held_tiles(c, seed)[0] * TILE - c["Lq"]
    else:
        st["Q"] = _normal((c["B"], c["Hq"], D), _dtype(c), _gen(seed, 0))
        if c["tail"] != "none":
            st["tail_k"], st["tail_v"], lens = _tail(c, seed)
            st["tail_len"] = lens.cuda() if c["tail"] == "rows" else int(lens[0])
        if c["entry"] != "plain":
            st["out"] = torch.empty_like(st["Q"])
            st["lse"] = torch.empty((c["B"], c["Hq"]), dtype=torch.float32, device="cuda")
        if c["entry"] == "kept":
            n = hb.decode_auto_splits(shape)
            st["workspace"] = torch.empty(hb.workspace_bytes(shape, 2, n + (c["tail"] != "none")), dtype=torch.uint8, device="cuda")
    return st


def _pools(kv):
    return {"k_dense": kv.k_dense, "k_nnz": kv.k_nnz, "k_meta": kv.k_meta, "k_map": kv.k_map,
            "v_dense": kv.v_dense, "v_nnz": kv.v_nnz, "v_meta": kv.v_meta, "v_map": kv.v_map}


def run(state):
    c, shape = state["case"], state["shape"]
    if c["op"] == "compress":
        return _pools(hb.compress_kv(shape, state["policy"], state["K"], state["V"]))
    kv = state["kv"]
    if c["op"] == "append":
        hb.append_tile(shape, kv, state["at"], state["K_new"], state["V_new"])
        return _pools(kv)
    if c["op"] == "recompress":
        return _pools(hb.recompress_kv(shape, kv, state["target"], counts=state["counts"]))
    if c["op"] == "prefill":
        return hb.prefill_attn(shape, state["Q"], kv, q_start=state["q_start"])
    if c["entry"] == "static":
        return hb.decode_attn_static(shape, state["Q"], kv, out=state["out"], lse=state["lse"])
    kept = dict(out=state["out"], lse=state["lse"], workspace=state["workspace"]) if c["entry"] == "kept" else {}
    if c["tail"] != "none":
        kept.update(tail_k=state["tail_k"], tail_v=state["tail_v"], tail_len=state["tail_len"])
    return hb.decode_attn(shape, state["Q"], kv, **kept)


# ------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------------------------
def _counts(c, held):
    """Tiles of a row that holds `held` tiles: kept, 2:4 K, 2:4 V."""
    prot = min(held, c["first"] + c["last"])
    kept = (held - prot) - int(c["skip"] * (held - prot))
    if _explicit(c):
        return held, (held - prot) * (c["sk"] >= 0.5), (held - prot) * (c["sv"] >= 0.5)
    return prot + kept, int(c["sk"] * kept), int(c["sv"] * kept)


def _tile_bytes(kept, nk, nv):
    return (2 * kept - nk - nv) * 16384 + (nk + nv) * 9216


def work(case):
    c = dict(case)
    T, rows = c["L"] // TILE, c["B"] * c["Hkv"]
    maps = 8 * T * rows
    held = _held_tiles(c, 1)
    packed = sum(c["Hkv"] * _tile_bytes(*_counts(c, n)) for n in held)
    if c["op"] == "compress":
        return {"bytes": 2.0 * rows * c["L"] * D * 2 + packed + maps, "flops": 0.0}
    if c["op"] == "append":
        n = max(1, c["n_new"])
        return {"bytes": rows * n * (2.0 * 16384 + 2 * 9216 + 8) + maps, "flops": 0.0}
    if c["op"] == "recompress":
        after = rows * _tile_bytes(*_counts(dict(c, sk=1.0, sv=1.0), T))
        return {"bytes": float(packed + after + 2 * maps), "flops": 0.0}
    if c["op"] == "decode":
        qo = 2 * c["B"] * c["Hq"] * D * 2 + 4 * c["B"] * c["Hq"]
        tail = 0 if c["tail"] == "none" else rows * 2 * TILE * D          # half a tail tile of K and V on average
        return {"bytes": float(packed + maps + qo + tail), "flops": 0.0}
    kept, nk, nv = _counts(c, held[0])
    end, Lq = held[0] * TILE, c["Lq"]
    pairs = c["B"] * c["Hq"] * Lq * (end - Lq + (Lq + 1) / 2.0) * kept / held[0]
    flops = 2.0 * D * pairs * ((1 - 0.5 * nk / kept) + (1 - 0.5 * nv / kept))   # a 2:4 tile takes half of the products
    return {"bytes": float(packed + maps + 2 * c["B"] * c["Hq"] * Lq * D * 2 + 4 * c["B"] * c["Hq"] * Lq), "flops": flops}


def tolerance(case):
    """Packed bytes and maps: every one.  Attention: four times what the same call shows with its sums in another order and
    against 64 bits, which is mostly the rounding of O to its 16 bits (8 resp. 11 significant ones)."""
    if case["op"] in ("compress", "append", "recompress"):
        return "exact"
    return {"rel": 6e-3} if case["dtype"] == "bf16" else {"rel": 1.2e-3}


# ------------------------------------------------------------------------------------------------------------------
# the same in 64 bits, from plain torch
# ------------------------------------------------------------------------------------------------------------------
def _keep2(x):
    """x [..., 4, n]: keep mask of the two largest magnitudes among the four, ties to the lower position."""
    mag = (x.contiguous().view(torch.int16).to(torch.int32) & 0x7FFF).unbind(-2)
    keep = []
    for i in range(4):
        above = sum(((mag[j] >= mag[i]) if j < i else (mag[j] > mag[i])).to(torch.int8) for j in range(4) if j != i)
        keep.append(above < 2)
    return torch.stack(keep, dim=-2)


def _mask_k(K):      # groups of 4 channels of a token
    return _keep2(K.reshape(K.shape[0], D // 4, 4, 1)).reshape(K.shape)


def _mask_v(V):      # groups of 4 tokens of a channel
    return _keep2(V.reshape(V.shape[0] // 4, 4, D)).reshape(V.shape)


def _row_states(c, K, V, mk, mv, held):
    """Tile states (0 skipped, 1 dense, 2 2:4) of one (batch, kv head) row, K, V [L, D]."""
    T = K.shape[0] // TILE
    if _explicit(c):
        sk, sv = _held_states(dict(c, B=1, Hkv=1), [held])
        return sk[0, 0].tolist(), sv[0, 0].tolist()
    first = min(c["first"], T)
    last = min(c["last"], T - first)
    mid = list(range(first, T - last))
    sk, sv = [1] * T, [1] * T

    def tiles(x):
        return x.reshape(T, -1).sum(1).tolist()

    n_skip = int(math.floor(c["skip"] * len(mid)))
    if n_skip:
        e = tiles(K.double() ** 2 + V.double() ** 2)
        for t in sorted(mid, key=lambda t: (e[t], t))[:n_skip]:
            sk[t] = sv[t] = 0
    kept = [t for t in mid if sk[t]]
    for s, X, m, f in ((sk, K, mk, c["sk"]), (sv, V, mv, c["sv"])):
        n = int(math.floor(f * len(kept)))
        if n:
            loss = tiles((X.double() * ~m).abs()) if n < len(kept) else [0.0] * T
            for t in sorted(kept, key=lambda t: (loss[t], t))[:n]:
                s[t] = 2
    return sk, sv


def exact(case, seed):
    c = dict(case)
    if c["op"] not in ("decode", "prefill"):
        return None                                          # bytes and whole numbers
    held = _held_tiles(c, seed)
    G = c["Hq"] // c["Hkv"]
    K, V = _kv_tensor(c, seed, 1, c["L"], c["outliers"]), _kv_tensor(c, seed, 2, c["L"], False)
    Lq = c["Lq"] if c["op"] == "prefill" else 1
    Q = _normal((c["B"], c["Hq"], Lq, D) if c["op"] == "prefill" else (c["B"], c["Hq"], D), _dtype(c), _gen(seed, 0))
    Q = Q.reshape(c["B"], c["Hq"], Lq, D)
    tail = _tail(c, seed) if c.get("tail", "none") != "none" else None
    O = torch.zeros((c["B"], c["Hq"], Lq, D), dtype=torch.float64, device="cuda")
    LSE = torch.full((c["B"], c["Hq"], Lq), -math.inf, dtype=torch.float64, device="cuda")
    for b in range(c["B"]):
        for h in range(c["Hkv"]):
            k, v = K[b, h], V[b, h]
            mk, mv = _mask_k(k), _mask_v(v)
            sk, sv = (torch.tensor(s, device="cuda").repeat_interleave(TILE) for s in _row_states(c, k, v, mk, mv, held[b]))
            at = torch.nonzero(sk != 0).reshape(-1)          # positions of the tokens that are kept
            k = (k.double() * (mk | (sk != 2)[:, None]))[at]
            v = (v.double() * (mv | (sv != 2)[:, None]))[at]
            if tail is not None:
                n = int(tail[2][b])
                k, v = torch.cat([k, tail[0][b, h, :n].double()]), torch.cat([v, tail[1][b, h, :n].double()])
            q0 = held[b] * TILE - Lq                         # position of the first query (prefill)
            step = max(64, int(1.5e8 // max(1, k.shape[0])))
            for hq in range(h * G, (h + 1) * G):
                for i in range(0, Lq, step):
                    q = Q[b, hq, i:i + step].double()
                    s = torch.matmul(q, k.t()) * (1.0 / math.sqrt(D))
                    if c["op"] == "prefill":
                        s.masked_fill_(at[None, :] > (q0 + i + torch.arange(q.shape[0], device="cuda"))[:, None], -math.inf)
                    lse = torch.logsumexp(s, dim=1)
                    seen = lse > -math.inf
                    p = torch.exp(s - torch.where(seen, lse, torch.zeros_like(lse))[:, None])
                    O[b, hq, i:i + step] = torch.matmul(p, v)
                    LSE[b, hq, i:i + step] = lse
    if c["op"] == "decode":
        return [O[:, :, 0], LSE[:, :, 0]]
    return [O, LSE]
