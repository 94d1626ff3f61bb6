"""The binding's native argument marshalling against the checks written out in Python: what it takes gives the same bits as the call
through ctypes, what it does not take raises what the Python checks raise."""
from __future__ import annotations

import pytest
import torch

from paper_2512_14481_amd import binding as B

CALLS = list(B._NATIVE)


def arguments(name, dev):
    """Valid arguments of entry point `name` on device `dev` and the positions of its outputs."""
    g = torch.Generator().manual_seed(5)
    M, N, K = 5, 32, 64

    def r(*shape, dtype=torch.float16):
        return torch.randn(shape, generator=g).to(dtype).to(dev)

    def z(*shape, dtype=torch.float16):
        return torch.zeros(shape, dtype=dtype, device=dev)

    f32, u8 = torch.float32, torch.uint8
    x, y, dy, s, ds = r(M, K), z(M, K), r(M, K), z(1, dtype=f32).add_(0.02), z(1, dtype=f32)
    s_k, ds_k = z(K, dtype=f32).add_(0.02), z(K, dtype=f32)
    w, s_w, out = torch.randint(-128, 128, (N, K), generator=g).to(torch.int8).to(dev), z(N, dtype=f32).add_(1e-3), z(M, N)
    if dev == "cpu":
        ws = z(1 << 16, dtype=u8)
    else:
        ws = B.new_workspace(1 << 16)
    lin = (x, s, w, s_w, None, out)
    wt = z(B.sasq_bwd_weight_bytes(N, K), dtype=u8)
    return {
        "sasq_fakequant_fwd": ((x, s, y, z(M, K, dtype=torch.int8), 8), (2, 3)),
        "sasq_fakequant_bwd": ((x, dy, s, y, ds, ws, 8), (3, 4)),
        "sasq_fakequant_fwd_batch": (([(x, s, y)], 8), (0,)),
        "sasq_fakequant_bwd_batch": (([(x, dy, s, y, ds)], ws, 8), (0,)),
        "sasq_fakequant_fwd_pc_batch": (([(x, s_k, y)], 8), (0,)),
        "sasq_fakequant_bwd_pc_batch": (([(x, dy, s_k, None, ds_k)], ws, 8), (0,)),
        "sasq_scale_sgd": ((s, r(1, dtype=f32), 0.1), (0,)),
        "sasq_scale_sgd_vec": ((s_k, r(K, dtype=f32), 0.1), (0,)),
        "sasq_scale_adamw": ((s_k, r(K, dtype=f32), ds_k, z(K, dtype=f32), 1, 0.1, 0.9, 0.99, 1e-8, 0.01), (0, 2, 3)),
        "sasq_static_linear": (lin + (B.SASQ_W_INT8, ws, z(M, N, dtype=torch.int32), z(M, K, dtype=torch.int8), 8), (5, 8, 9)),
        "sasq_static_linear_batch": (([lin], B.SASQ_W_INT8, ws, 8), (0,)),
        "sasq_static_linear_grouped": ((x, s_k[:2].clone(), w, s_w, r(N, dtype=f32), out, 32, B.SASQ_W_INT8, ws, z(M, N, dtype=f32), None, 8), (5, 9)),
        "sasq_linear_bwd_input": ((r(M, N), wt.view(torch.float16).normal_(generator=None).view(u8), y, K, z(M, K, dtype=f32)), (2, 4)),
        "sasq_absmax_scale": ((x, s, ws, 8), (1,)),
        "sasq_quantize_weight": ((r(N, K, dtype=f32), w, s_w, B.SASQ_W_INT8), (1, 2)),
        "sasq_pack_weight": ((w, z(B.sasq_packed_weight_bytes(N, K, B.SASQ_W_INT8_BLOCKED), dtype=u8), N, K, B.SASQ_W_INT8), (1,)),
        "sasq_prepare_bwd_weight": ((w, s_w, wt, N, K, B.SASQ_W_INT8, torch.float16), (2,)),
    }[name]


def native(name, args):
    args = list(args)
    if name == "sasq_prepare_bwd_weight":
        args[6] = B._DT.get(args[6])
    return getattr(B._native, name)(*args)


def broken(args):
    """The arguments with one thing wrong each: a tensor on the other device's side, not contiguous, of another type, cut short; an item short."""
    for i, a in enumerate(args):
        if isinstance(a, list):
            for item in broken(a[0]):
                yield args[:i] + ([item],) + args[i + 1:]
            yield args[:i] + ([],) + args[i + 1:]
            yield args[:i] + (a * (B.SASQ_MAX_BATCH + 1),) + args[i + 1:]
        elif isinstance(a, torch.Tensor):
            wide = torch.empty(tuple(a.shape) + (2,), dtype=a.dtype, device=a.device)[..., 0]
            for bad in (a.cpu(), wide, a.to(torch.float64), a.reshape(-1)[:-1] if a.numel() > 1 else a.to(torch.int16)):
                yield args[:i] + (bad,) + args[i + 1:]


@pytest.mark.parametrize("name", CALLS)
def test_host_tensors_and_odd_arguments_are_left_to_the_checks(name):
    B._lib()
    args, _ = arguments(name, "cpu")
    assert native(name, args) is None
    assert getattr(B._native, name)() is None and getattr(B._native, name)(*([None] * len(args))) is None
    with pytest.raises(ValueError, match="device tensors"):
        getattr(B, name)(*args)


def outputs(args, where):
    for i in where:
        if isinstance(args[i], list):
            yield from (t for t in args[i][0] if isinstance(t, torch.Tensor))
        elif args[i] is not None:
            yield args[i]


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
def test_same_bits_and_same_errors_as_through_ctypes(name, monkeypatch):
    B._lib()
    fast = B._native

    def run():
        torch.manual_seed(3)
        args, where = arguments(name, "cuda")
        assert getattr(B, name)(*args) is None
        torch.cuda.synchronize()
        return [t.clone() for t in outputs(args, where)]

    torch.manual_seed(3)
    assert native(name, arguments(name, "cuda")[0]) == 0            # taken, not left to the checks
    got = run()
    monkeypatch.setattr(B, "_native", B._Unbound())
    want = run()
    assert len(got) == len(want) and all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, want))

    def error(args):
        try:
            getattr(B, name)(*args)
        except Exception as e:                                      # noqa: BLE001 -- compared below
            return type(e), str(e)
        return None

    for args in broken(arguments(name, "cuda")[0]):
        by_ctypes = error(args)
        if by_ctypes is None:
            continue                                                # taken as it is: a length that no check looks at
        with monkeypatch.context() as m:
            m.setattr(B, "_native", fast)
            assert error(args) == by_ctypes


@pytest.mark.parametrize("how", ["missing", "not a module", "built for another torch"])
def test_without_the_native_module_the_calls_go_through_ctypes(how, monkeypatch, tmp_path):
    if how == "built for another torch":
        monkeypatch.setattr(B, "marshal_abi", lambda: "torch 0.0")
    else:
        monkeypatch.setattr(B, "MARSHAL_PATH", str(tmp_path / "_marshal.so"))
        if how == "not a module":
            (tmp_path / "_marshal.so").write_text("no library")
    monkeypatch.setattr(B, "_LIB", None)
    monkeypatch.setattr(B, "_native", B._Unbound())
    with pytest.warns(RuntimeWarning, match="go through ctypes"):
        assert B.sasq_version() >= 100
    for name in CALLS:
        args, _ = arguments(name, "cpu")
        assert native(name, args) is None
        with pytest.raises(ValueError, match="device tensors"):                # the checks written out in Python
            getattr(B, name)(*args)
