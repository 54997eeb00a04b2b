"""csrc/marshal.cpp: it answers None to whatever is not an ordinary call (the binding's own path then says what is wrong), and what it
takes ends as the same C call: same bits, same error codes, as with marshalling in Python."""
import ctypes
import shutil

import numpy as np
import pytest
import torch

import paper_2605_14217_amd as preft
from paper_2605_14217_amd import binding
from paper_2605_14217_amd import workloads as wl


@pytest.fixture
def native():
    preft.load_library()
    assert binding._native is not None, "_marshal.so is not built"
    return binding._native


def test_what_is_no_ordinary_call_goes_through_the_binding(native):
    t = torch.zeros(4, 8)
    i32, i64 = torch.zeros(3, dtype=torch.int32), torch.zeros(2, dtype=torch.int64)
    ws = torch.zeros(64, dtype=torch.uint8)
    rest = (4, 1.0, 0, ws, 0, 0)
    assert native.lora(t, t, i32, i32, i32, i64, i64, *rest) is None                 # host tensors
    assert native.lora(t, None, i32, i32, i32, i64, i64, *rest) is None
    assert native.lora(t) is None and native.schedule() is None and native.reft(False) is None
    assert native.lora_packed([], t, i32, i32, i32, [], [], *rest) is None
    assert native.reft_layers([], i64, i32, i32, i32, i64, i64, None, 2, *rest) is None
    with pytest.raises(ValueError, match="y: need a 2-D device tensor"):
        preft.preft_lora_apply(t, t, i32, i32, i32, i64, i64, 4, 1.0, 0, ws, stream=0)
    with pytest.raises(ValueError, match="seg_start"):
        preft.preft_schedule(ws, i32, i32, i32, 4, 2, 0, stream=0)
    if not torch.cuda.is_available():                         # nor does asking for the current stream come before the checks
        with pytest.raises(ValueError, match="y: need a 2-D device tensor"):
            preft.preft_lora_apply(t, t, i32, i32, i32, i64, i64, 4, 1.0, 0, ws)
        with pytest.raises(ValueError, match=r"ys\[0\]|x: need a 2-D device tensor"):
            preft.preft_lora_apply_packed([t], t, i32, i32, i32, [i64], [i64], 4, 1.0, 0, ws)
        with pytest.raises(ValueError, match="h: need a 2-D device tensor"):
            preft.preft_direft_apply(t, i32, i32, i32, i64, i64, None, 4, 1.0, 0, ws)
        with pytest.raises(ValueError, match=r"hs\[0\]: need a 2-D device tensor"):
            preft.preft_direft_apply_layers([t], i64, i32, i32, i32, i64, i64, None, 2, 4, 1.0, 0, ws)
        with pytest.raises(ValueError, match="seg_start"):
            preft.preft_schedule(ws, i32, i32, i32, 4, 2, 0)
    with pytest.raises(TypeError):
        native.bind(1, 2)


def test_a_module_built_for_another_torch_is_not_used(native, monkeypatch):
    """It reads tensors at the offsets of the torch and Python that it was compiled against: any other pair goes without it."""
    from paper_2605_14217_amd import build
    assert native.built_for() == build.built_for() and torch.__version__ in native.built_for()
    monkeypatch.setattr(torch, "__version__", torch.__version__ + "x")
    with pytest.warns(UserWarning, match="was built for"):
        assert binding._load_marshal(binding._lib) is None


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("command", [["/nonexistent/g++"], ["g++", "/nonexistent.cpp"], None], ids=["no compiler", "does not compile", "no torch headers"])
def test_the_library_is_built_without_the_module(command, tmp_path, monkeypatch):
    """What keeps _marshal.so from being built keeps neither libpreft.so from it nor an older module in place."""
    from paper_2605_14217_amd import build
    src = tmp_path / "one.hip"
    src.write_text('#include <hip/hip_runtime.h>\nextern "C" int one() { return 1; }\n')

    def no_headers(out):
        raise ImportError("torch.utils.cpp_extension")
    monkeypatch.setattr(build, "sources", lambda: [str(src)])
    monkeypatch.setattr(build, "LIB_PATH", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
    monkeypatch.setattr(build, "marshal_command", no_headers if command is None else lambda out: command)
    (tmp_path / "_marshal.so").write_text("older")
    with pytest.warns(UserWarning, match="not built"):
        assert build.build_library() == str(tmp_path / "lib.so")
    assert ctypes.CDLL(str(tmp_path / "lib.so")).one() == 1 and not (tmp_path / "_marshal.so").exists()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_same_calls_as_the_python_path(native, dtype, monkeypatch):
    from parity_util import bits, dev_tables, direft_pools_to_device, lora_pools_to_device
    N, r, d = 3, 8, 256
    lens = np.array([40, 1, 1, 17, 1])
    tab = wl.from_lengths(lens, np.array([0, 1, 2, 2, -1]), np.where(lens > 1, lens, 0))
    ss, sa, sp = dev_tables(tab)
    x, h0, y0 = (wl.activations(tab.T, n, dtype, device="cuda", seed=n) for n in (d, d + 8, 2 * d))
    A, B, keep = lora_pools_to_device(wl.lora_pool(N, r, d, d, dtype, device="cuda", seed=1))
    dp = wl.direft_pool(N, r, d + 8, dtype, device="cuda", seed=2)
    W1, W2t, b, keep2 = direft_pools_to_device(dp)

    def step(stream):
        ws = preft.new_workspace(tab.T, tab.S, z_rank=r, z_proj=2)
        y, h, l = y0.clone(), h0.clone(), h0.clone()
        ls = [h0.clone(), h0.clone()]
        tables = [torch.tensor([t.data_ptr()] * 2, dtype=torch.int64, device="cuda") for t in (W1, W2t, b)]
        mode, ready = preft.PREFT_ALL_TOKENS, preft.PREFT_ALL_TOKENS | preft.PREFT_SCHEDULE_READY
        preft.preft_schedule(ws, ss, sa, sp, tab.T, N, mode, stream)
        preft.preft_lora_apply(y[:, :d], x, ss, sa, sp, A, B, r, 2.0, ready, ws, stream)
        preft.preft_lora_apply_packed((y[:, :d], y[:, d:]), x, ss, sa, sp, [A, A], (B, B), r, 0.5, ready, ws, stream)
        preft.preft_direft_apply(h, ss, sa, sp, W1, W2t, b, r, 0.5, ready, ws, stream)
        preft.preft_loreft_apply(l, ss, sa, sp, W1, W2t, None, r, 1, ready, ws, stream)              # an int as scale
        preft.preft_direft_apply_layers(ls, preft.pointer_table(ls), ss, sa, sp, *tables, N, r, 0.5, ready, ws, stream)
        codes = []
        for bad in (dict(rank=0), dict(rank=500), dict(mode=0x8000)):
            with pytest.raises(preft.PreftError) as e:
                preft.preft_lora_apply(y[:, :d], x, ss, sa, sp, A, B, bad.get("rank", r), 2.0, bad.get("mode", ready), ws, stream)
            codes.append((e.value.code, str(e.value)))
        with pytest.raises(ValueError, match="equal length"):
            preft.preft_lora_apply(y[:, :d], x, ss, sa, sp, A, B[:1], r, 2.0, ready, ws, stream)
        with pytest.raises(ValueError, match="unit column stride"):
            preft.preft_direft_apply(h.t(), ss, sa, sp, W1, W2t, b, r, 0.5, ready, ws, stream)
        torch.cuda.synchronize()
        return [y, h, l] + ls, codes

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    got = [step(None), step(side)]
    monkeypatch.setattr(binding, "_native", None)
    want, codes = step(None)
    for tensors, c in got:
        assert c == codes and all(torch.equal(bits(a), bits(w)) for a, w in zip(tensors, want))
    assert not torch.equal(bits(want[0]), bits(y0))


@pytest.mark.gpu
def test_slot_pools_and_numbers_of_other_types_are_marshalled_too(native):
    """The slot manager's pools, NumPy integers and whole-number scales: one native call each (an answer that is not None), with the bits of
    the ordinary call; a pool of another length is declined."""
    from parity_util import bits, dev_tables
    N, r, d = 3, 8, 256
    tab = wl.from_lengths(np.array([40, 1, 17]), np.array([0, 1, 2]), np.array([40, 1, 17]))
    seg = dev_tables(tab)
    x, y0 = (wl.activations(tab.T, n, "bf16", device="cuda", seed=n) for n in (d, d + 8))
    pool = wl.lora_pool(N, r, d, d + 8, "bf16", device="cuda", seed=1)
    host = [[t.cpu().contiguous() for t in part] for part in (pool.A, pool.B)]
    stream = torch.cuda.current_stream().cuda_stream
    ws = preft.new_workspace(tab.T, tab.S)
    mgr = preft.preft_slots_create(N, N, [r * d * 2, (d + 8) * r * 2])
    try:
        for a in range(N):
            for part in range(2):
                preft.preft_slots_store(mgr, a, part, host[part][a])
        slots = preft.preft_slots_acquire(mgr, list(range(N)))
        refs = [preft.preft_slots_pool(mgr, part) for part in range(2)]
        order = sorted(range(N), key=lambda a: slots[a])       # slot -> adapter
        tables = [preft.pointer_table([m[a].contiguous() for a in order]) for m in (pool.A, pool.B)]
        got = []
        for A, B, rank, scale, mode in ((*tables, r, 2.0, preft.PREFT_ALL_TOKENS), (*refs, r, 2.0, preft.PREFT_ALL_TOKENS), (refs[0], tables[1], np.int64(r), 2, np.int32(1)),
                                        (*tables, np.int32(r), np.float32(2.0), True)):
            y, z = y0.clone(), y0.clone()
            assert native.lora(y, x, *seg, A, B, rank, scale, mode, ws, stream, 0) == 0
            assert native.lora_packed([z], x, *seg, [A], [B], rank, scale, mode, ws, stream, 0) == 0
            got += [y, z]
        h, l = x.clone(), x.clone()
        square = binding.PoolRef(refs[0].data_ptr(), N)          # [r, d] matrices as both factors: any bytes will do
        assert native.reft(False, h, *seg, square, square, None, r, 1, preft.PREFT_ALL_TOKENS, ws, stream, 0) == 0
        assert native.reft(False, l, *seg, tables[0], square, None, r, 1.0, preft.PREFT_ALL_TOKENS, ws, stream, 0) == 0
        assert native.schedule(ws, *seg, np.int64(tab.T), N, 1, stream) == 0
        assert native.lora(y0, x, *seg, refs[0], binding.PoolRef(refs[1].data_ptr(), N - 1), r, 2.0, 1, ws, stream, 0) is None
        assert native.lora(y0, x, *seg, *refs, 2.5, 2.0, 1, ws, stream, 0) is None and native.lora(y0, x, *seg, *refs, r, "2", 1, ws, stream, 0) is None
        assert native.lora(y0, x, *seg, *refs, 1 << 40, 2.0, 1, ws, stream, 0) is None
        torch.cuda.synchronize()
        assert all(torch.equal(bits(v), bits(got[0])) for v in got) and torch.equal(bits(h), bits(l)) and not torch.equal(bits(got[0]), bits(y0))
    finally:
        torch.cuda.synchronize()
        preft.preft_slots_destroy(mgr)
