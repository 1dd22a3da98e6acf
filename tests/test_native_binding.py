"""The native part of the binding against the binding's own Python code: the same calls through both give the same bits, and
whatever the native part does not take as it is goes on to the Python code, which accepts or refuses it as before."""
import collections
import sys
import threading
import time
import types

import pytest
import torch

from paper_2604_16864_amd import binding as hb


class _PythonOnly:
    """Leaves every call to the Python code."""

    def __getattr__(self, name):
        return lambda *a: None


class _Recorder:
    """Notes which native functions are called and whether each took its call."""

    def __init__(self, native):
        self.native, self.calls = native, []

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self.native, name)(*args)
            self.calls.append((name, r is not None))
            return r
        return call


def _shape(dtype=hb.BF16):
    return hb.make_shape(2, 8, 2, 64 * 12, dtype=dtype)


def test_calls_the_native_part_leaves_alone_are_refused_as_before():
    hb.lib()
    sh = _shape()
    kv = hb.PackedKV(sh, [0, 0, 12, 0, 12], "cpu")
    q = torch.zeros(2, 8, 128, dtype=torch.bfloat16)
    bad = [q,                                                     # not on the GPU
           q.to(torch.float16), q.float(), q.transpose(0, 1)]
    for t in bad:
        with pytest.raises(AssertionError):
            hb.decode_attn(sh, t, kv)
        with pytest.raises(AssertionError):
            hb.decode_attn_static(sh, t, kv, out=torch.empty_like(q))
        with pytest.raises(AssertionError):
            hb.prefill_attn(sh, t[:, :, None], kv)
    tile = torch.zeros(2, 2, 64, 128, dtype=torch.bfloat16)
    for k, v in ((tile[:, :, :63], tile[:, :, :63]), (tile.float(), tile.float()), (tile, tile.transpose(0, 1)), (tile[:1], tile[:1])):
        with pytest.raises(AssertionError):
            hb.append_tile(sh, kv, 0, k, v)
    with pytest.raises(AttributeError):
        hb.decode_attn(sh, q.tolist(), kv)
    n = hb._fast()
    assert n.decode(sh, q, kv, 0.0, 0, True, None, None, None, None, None, None) is None
    assert n.decode(sh, q, object(), 0.0, 0, True, None, None, None, None, None, None) is None
    assert n.decode(q, q, kv, 0.0, 0, True, None, None, None, None, None, None) is None
    k = torch.zeros(2, 2, 768, 128, dtype=torch.bfloat16)
    for a, b in ((k, k), (k.float(), k.float()), (k, k.transpose(0, 1)), (k[..., ::2], k[..., ::2])):
        with pytest.raises(AssertionError):
            hb.compress_kv(sh, hb.make_policy(), a, b)
    assert n.compress(sh, hb.make_policy(), k, k) is None and n.compress(sh, sh, k, k) is None
    assert n.recompress(sh, kv, hb.make_policy(), (0, 0, 12, 0, 12), None) is None
    assert n.prefill() is None and n.append(1, 2) is None and n.pools(sh, [0, 0, 12, 0], q) is None


@pytest.mark.parametrize("counts", [[0, 0, 12, 0, 12], [0, 12, 0, 5, 7], [3, 9, 0, 0, 9]])
def test_pools_made_natively_are_the_same(counts):
    sh = _shape()
    a, b = hb.PackedKV(sh, counts, "cpu", torch.empty(1)), hb.PackedKV(sh, counts, "cpu")
    assert (a.nbytes, a.counts, a.uniform) == (b.nbytes, b.counts, b.uniform)
    for name in ("k_dense", "k_nnz", "k_meta", "k_map", "v_dense", "v_nnz", "v_meta", "v_map"):
        x, y = getattr(a, name), getattr(b, name)
        assert (x is None) == (y is None)
        assert x is None or (x.shape == y.shape and x.dtype == y.dtype and x.device == y.device)


@pytest.mark.parametrize("how", ["another torch", "not built", "of before"])
def test_without_a_native_part_that_fits_calls_go_through_python(how, monkeypatch):
    """A native part that was built against another torch, or none at all, is left alone with a warning; the library works."""
    hb.lib()
    name = "paper_2604_16864_amd._hs_torch"
    other = types.ModuleType(name)
    other.bind = lambda *a: pytest.fail("a module of another torch was used")
    if how == "another torch":
        other.built_for = sys.modules[name].built_for.replace("torch ", "torch 1")
    monkeypatch.setitem(sys.modules, name, None if how == "not built" else other)       # None: the import fails
    monkeypatch.delattr(sys.modules["paper_2604_16864_amd"], "_hs_torch", raising=False)
    monkeypatch.setattr(hb, "_lib", None)
    monkeypatch.setattr(hb, "_native", None)
    with pytest.warns(RuntimeWarning, match="native part"):
        sh = _shape()
        assert hb.tile_counts(sh, hb.make_policy()) == [0, 0, 12, 0, 12]
    kv = hb.PackedKV(sh, [0, 0, 12, 0, 12], "cpu", torch.empty(1))
    assert kv.nbytes == sum(hb.kv_bytes(sh, kv.counts)) and kv.k_nnz.device.type == "cpu"
    q = torch.zeros(2, 8, 128, dtype=torch.bfloat16)
    for call in (lambda: hb.decode_attn(sh, q, kv), lambda: hb.decode_attn_static(sh, q, kv, out=q), lambda: hb.prefill_attn(sh, q[:, :, None], kv),
                 lambda: hb.append_tile(sh, kv, 0, q, q), lambda: hb.compress_kv(sh, hb.make_policy(), q, q)):
        with pytest.raises((AssertionError, IndexError)):
            call()


def test_the_native_part_is_used_where_it_fits():
    hb.lib()
    assert type(hb._native) is types.ModuleType and hb._native.built_for.startswith(f"torch {torch.__version__}, Python 3")
    assert all(callable(getattr(hb._native, name)) for name in hb._NATIVE_CALLS)


def test_other_threads_run_while_the_native_part_allocates():
    """An allocation may wait for the GPU, and the GPU for what another thread has yet to do.  Made slow here by torch's option that
    fills new memory."""
    sh = hb.make_shape(1, 8, 8, 64 * 4096)
    like, ticks, stop = torch.empty(1), [], threading.Event()
    pools = hb._fast().pools

    def tick():
        while not stop.wait(0.001):
            ticks.append(time.perf_counter())
    before, n = torch.are_deterministic_algorithms_enabled(), torch.get_num_threads()
    t = threading.Thread(target=tick)
    t.start()
    try:
        torch.use_deterministic_algorithms(True)
        torch.set_num_threads(1)                               # 1 GB by one thread: far above the 5 ms after which threads change
        t0 = time.perf_counter()
        bufs = pools(sh, [0, 4096, 0, 4096, 0], like)
        t1 = time.perf_counter()
    finally:
        torch.set_num_threads(n)
        torch.use_deterministic_algorithms(before)
        stop.set()
        t.join()
    assert bufs is not None
    assert any(t0 + 0.25 * (t1 - t0) < x < t1 - 0.25 * (t1 - t0) for x in ticks)


def test_an_allocation_that_fails_is_raised():
    with pytest.raises(RuntimeError, match="alloc"):
        hb._fast().pools(hb.make_shape(4096, 8, 8, 64 << 24), [0, 1 << 24, 0, 1 << 24, 0], torch.empty(1))     # beyond any address space


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("policy", [dict(), dict(sparse_frac_k=0.5, skip_frac=0.25)])
def test_native_and_python_calls_give_the_same_bits(dtype, policy, monkeypatch):
    sh = hb.make_shape(2, 8, 2, 64 * 12, dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(5)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=g).to(dtype)
    K, V, q, Q, tk, tv = (normal(*s) for s in ((2, 2, 768, 128), (2, 2, 768, 128), (2, 8, 128), (2, 8, 128, 128), (2, 2, 64, 128),
                                               (2, 2, 64, 128)))
    lens = torch.tensor([7, 64], dtype=torch.int32, device="cuda")
    old = torch.tensor([4, 9], dtype=torch.int32, device="cuda")
    ws = torch.empty(hb.workspace_bytes(sh, 2, 5), dtype=torch.uint8, device="cuda")

    def calls():
        kv = hb.compress_kv(sh, hb.make_policy(**policy), K, V)
        held = dict(out=torch.empty_like(q), lse=torch.empty(2, 8, device="cuda"))
        yield hb.decode_attn(sh, q, kv)
        yield hb.decode_attn(sh, q, kv, scale=1, n_splits=3, want_lse=False)
        yield hb.decode_attn(sh, q, kv, n_splits=4, workspace=ws, tail_k=tk, tail_v=tv, tail_len=33, **held)
        yield hb.decode_attn(sh, q, kv, tail_k=tk, tail_v=tv, tail_len=lens)
        yield hb.decode_attn(sh, q, kv, tail_len=0)
        yield hb.decode_attn_static(sh, q, kv, out=torch.empty_like(q), lse=torch.empty(2, 8, device="cuda"))
        yield hb.prefill_attn(sh, Q, kv)
        yield hb.prefill_attn(sh, Q, kv, causal=False, scale=0.1, want_lse=False, q_start=192)
        yield hb.prefill_attn(sh, torch.nn.Parameter(Q), kv, q_start=64)
        sk = torch.zeros(2, 2, 12, dtype=torch.int8)
        sk[:, :, :4] = hb.SPARSE24
        grow = hb.compress_kv(sh, hb.make_policy(state_k=sk.numpy(), state_v=sk.numpy()), K, V,
                              out=hb.PackedKV(sh, [0, 2, 12, 2, 12], "cuda"))
        hb.append_tile(sh, grow, old, tk, tv)
        hb.append_tile(sh, grow, 5, K[:, :, :128], V[:, :, :128], state_k=hb.DENSE)
        yield hb.unpack_kv(sh, grow)
        for made in (kv, hb.recompress_kv(sh, kv, hb.make_policy()), hb.recompress_kv(sh, kv, hb.make_policy(dense_first_tiles=2)),
                     hb.recompress_kv(sh, kv, hb.make_policy(sparse_frac_k=0.0), counts=[0, 12, 12, 12, 12])):
            yield hb.unpack_kv(sh, made)
            yield made.k_map, made.v_map, torch.tensor(made.counts + [made.uniform, made.nbytes])
    stream, record = torch.cuda.Stream(), _Recorder(hb._fast())
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream), monkeypatch.context() as m:
        m.setattr(hb, "_native", record)
        native = list(calls())
        stream.synchronize()
        took = collections.Counter(name for name, taken in record.calls if taken)
        assert all(taken for _, taken in record.calls)          # every call was the native part's
        assert took.pop("prefill") >= 3                         # twice where a call wants scratch
        assert took == dict(compress=1, decode=5, decode_static=1, append=2, recompress=3)
        record.calls.clear()                                    # what it leaves to the Python code, but for the new cache's buffers
        sk = torch.full((2, 2, 12), hb.SPARSE24, dtype=torch.int8, device="cuda")
        hb.compress_kv(sh, hb.make_policy(state_k=sk, state_v=sk), K, V)
        hb.recompress_kv(sh, hb.compress_kv(sh, hb.make_policy(), K, V), hb.make_policy(state_k=sk, state_v=sk))
        stream.synchronize()
        assert record.calls == [("compress", False), ("pools", True), ("compress", True), ("recompress", False), ("pools", True)]
    with monkeypatch.context() as m:
        m.setattr(hb, "_native", _PythonOnly())
        python = list(calls())
    torch.cuda.synchronize()
    assert len(native) == len(python)
    for i, (a, b) in enumerate(zip(native, python)):
        for x, y in zip(a, b):
            assert (x is None) == (y is None), i
            assert x is None or (type(x) is type(y) and x.dtype == y.dtype and torch.equal(x.view(torch.uint8), y.view(torch.uint8))), i


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_prefill_makes_its_outputs_before_it_takes_scratch(native, monkeypatch):
    """The call can do without scratch but not without its outputs: where memory holds one of them, they have it."""
    sh = hb.make_shape(1, 8, 2, 64 * 40)
    K = torch.randn(1, 2, sh.L, 128, device="cuda").to(torch.bfloat16)
    kv = hb.compress_kv(sh, hb.make_policy(), K, K)
    Q = torch.randn(1, 8, 64, 128, device="cuda").to(torch.bfloat16)
    assert hb.prefill_workspace_bytes(sh, 64, sh.L - 64, kv) > 0
    before, held = torch.cuda.memory_allocated(), []

    def none_left(nbytes, device):
        assert nbytes == hb.prefill_workspace_bytes(sh, 64, sh.L - 64, kv)      # what the call uses and no more
        held.append(torch.cuda.memory_allocated() - before)
        raise torch.OutOfMemoryError("no scratch to be had")
    monkeypatch.setattr(hb, "_workspace", none_left)
    if not native:
        monkeypatch.setattr(hb, "_native", _PythonOnly())
    for want_lse in (True, False):
        O, LSE = hb.prefill_attn(sh, Q, kv, want_lse=want_lse)
        assert held.pop() == torch.cuda.memory_allocated() - before >= O.nbytes + (LSE.nbytes if want_lse else 0) and (LSE is None) != want_lse
        assert torch.isfinite(O).all()
        del O, LSE


@pytest.mark.gpu
def test_library_errors_are_raised_through_the_native_part():
    sh = _shape()
    K = torch.zeros(2, 2, 768, 128, dtype=torch.bfloat16, device="cuda")
    kv = hb.compress_kv(sh, hb.make_policy(), K, K)
    q = torch.zeros(2, 8, 128, dtype=torch.bfloat16, device="cuda")
    for kw in (dict(n_splits=-1), dict(scale=-1.0)):
        with pytest.raises(hb.HsError):
            hb.decode_attn(sh, q, kv, **kw)
    for kw in (dict(tail_len=65), dict(tail_len=0, n_splits=2**31 - 1)):
        with pytest.raises(hb.HsError):
            hb.decode_attn(sh, q, kv, **kw)
    with pytest.raises(hb.HsError):
        hb.prefill_attn(sh, torch.zeros(2, 8, 100, 128, dtype=torch.bfloat16, device="cuda"), kv)
    for kw in (dict(skip_frac=2.0), dict(sparse_frac_k=-0.5), dict(dense_first_tiles=-1)):
        with pytest.raises(hb.HsError):
            hb.compress_kv(sh, hb.make_policy(**kw), K, K)
        with pytest.raises(hb.HsError):
            hb.recompress_kv(sh, kv, hb.make_policy(**kw), counts=[0, 0, 12, 0, 12])
    with pytest.raises(hb.HsError):                              # ranks tiles, without scores
        hb.recompress_kv(sh, kv, hb.make_policy(skip_frac=0.5))
    with pytest.raises(hb.HsError):                              # a uniform cache does not grow
        hb.append_tile(sh, kv, 3, torch.zeros(2, 2, 64, 128, dtype=torch.bfloat16, device="cuda"),
                       torch.zeros(2, 2, 64, 128, dtype=torch.bfloat16, device="cuda"))


@pytest.mark.gpu
def test_native_outputs_follow_the_modes_of_the_thread():
    """New tensors are made past the dispatcher only where nothing listens: inference mode, a dispatch mode, memory that is to be
    filled, and another stream give what the Python code gives."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        def __init__(self):
            super().__init__()
            self.names = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.names.append(str(func))
            return func(*args, **(kwargs or {}))

    sh = hb.make_shape(1, 4, 2, 256)
    g = torch.Generator(device="cuda").manual_seed(8)
    K, V = (torch.randn((1, 2, 256, 128), device="cuda", generator=g).bfloat16() for _ in range(2))
    q = torch.randn((1, 4, 128), device="cuda", generator=g).bfloat16()
    plain = hb.decode_attn(sh, q, hb.compress_kv(sh, hb.make_policy(), K, V))
    assert hb._native is not None
    assert not any(x.is_inference() or x.requires_grad for x in plain)
    assert plain[0].dtype == q.dtype and plain[0].device == q.device and plain[0].stride() == q.stride() and plain[1].shape == (1, 4)

    def same(pair):
        return all(torch.equal(x, y) for x, y in zip(pair, plain))
    with torch.inference_mode():
        kv = hb.compress_kv(sh, hb.make_policy(), K, V)
        out = hb.decode_attn(sh, q, kv)
        assert all(x.is_inference() for x in (*out, kv.k_map, kv.v_nnz))
    assert same(out)
    with Seen() as seen:
        out = hb.decode_attn(sh, q, hb.compress_kv(sh, hb.make_policy(), K, V))
    assert same(out) and sum("empty" in n for n in seen.names) >= 8
    torch.use_deterministic_algorithms(True)
    try:
        room = hb.PackedKV(sh, [0, 0, 6, 0, 6])                     # slots nobody writes
        assert torch.utils.deterministic.fill_uninitialized_memory and int(room.k_nnz.reshape(2, 6, -1)[:, 4:].min()) == 255
        kv = hb.compress_kv(sh, hb.make_policy(), K, V)
        more = hb.recompress_kv(sh, kv, hb.make_policy(), counts=[0, 0, 6, 0, 6])
        assert int(more.k_nnz.reshape(2, 6, -1)[:, 4:].min()) == 255
        assert same(hb.decode_attn(sh, q, kv))
    finally:
        torch.use_deterministic_algorithms(False)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        out = hb.decode_attn(sh, q, hb.compress_kv(sh, hb.make_policy(), K, V))
    side.synchronize()
    assert same(out)


@pytest.mark.gpu
def test_native_outputs_are_seen_by_observers():
    """A profiler sees the tensors that a call makes, as it sees those of the Python code; a call into kept buffers makes none."""
    sh = hb.make_shape(1, 4, 2, 256)
    K, V = (torch.ones((1, 2, 256, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    q, q4 = (torch.ones(n, dtype=torch.bfloat16, device="cuda") for n in ((1, 4, 128), (1, 4, 64, 128)))
    kv = hb.compress_kv(sh, hb.make_policy(), K, V)
    assert hb._native is not None
    room = torch.empty(hb.workspace_bytes(sh, 2, 0), dtype=torch.uint8, device="cuda")
    o, lse = hb.decode_attn(sh, q, kv)

    def made(call):
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as seen:
            call()
        return sum(e.name in ("aten::empty", "aten::empty_strided") for e in seen.events())
    assert made(lambda: hb.decode_attn(sh, q, kv)) == 3                              # O, LSE, scratch
    assert made(lambda: hb.prefill_attn(sh, q4, kv, want_lse=False)) == 1
    assert made(lambda: hb.compress_kv(sh, hb.make_policy(skip_frac=0.5), K, V)) == 7  # K and V: values, positions, map; scratch
    assert made(lambda: hb.decode_attn(sh, q, kv, out=o, lse=lse, workspace=room)) == 0


@pytest.mark.gpu
def test_native_outputs_have_the_strides_of_the_queries():
    """O is laid out as torch.empty_like lays it out, also where a batch of one is cut from a tensor with more heads."""
    sh = hb.make_shape(1, 4, 2, 256)
    K, V = (torch.ones((1, 2, 256, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    kv = hb.compress_kv(sh, hb.make_policy(), K, V)
    assert hb._native is not None
    for call, q in ((hb.decode_attn, torch.ones((1, 6, 128), dtype=torch.bfloat16, device="cuda")[:, :4]),
                    (hb.prefill_attn, torch.ones((1, 6, 64, 128), dtype=torch.bfloat16, device="cuda")[:, :4])):
        assert q.is_contiguous() and q.stride(0) == 6 * q[0, 0].numel()
        for kept in (dict(), dict(want_lse=False)):
            assert call(sh, q, kv, **kept)[0].stride() == torch.empty_like(q).stride() == q.stride()
