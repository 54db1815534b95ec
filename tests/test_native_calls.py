"""The native calls of the binding against its general code: same outputs, same refusals."""
import ctypes
import itertools
import struct
import threading

import pytest
import torch

from paper_2601_11660_amd import binding as B
from paper_2601_11660_amd import build


class General:
    """Stands in for the native calls and leaves every call to the general code."""

    def __getattr__(self, name):
        return lambda *a: None


@pytest.mark.parametrize("content", [None, b"not a library", b"\x7fELF"])
def test_the_binding_works_without_the_module(content, tmp_path, monkeypatch):
    """Missing or not loadable, it takes no entry point with it."""
    path = tmp_path / "_native.so"
    if content is not None:
        path.write_bytes(content)
    monkeypatch.setattr(B, "NATIVE_PATH", str(path))
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_calls", None)
    with pytest.warns(RuntimeWarning, match="does not load"):
        L = B.lib()
    assert B.lib() is L and B.packed_weights_bytes(64, 64) > 0
    for _, f, args in cases("cpu"):
        with pytest.raises(ValueError, match="expected a device tensor"):
            f(*args)


def test_a_build_without_a_host_compiler_leaves_no_module(tmp_path, monkeypatch, capsys):
    stale = tmp_path / "_native.so"
    stale.write_bytes(b"built for another torch")
    monkeypatch.setattr(build, "NATIVE", str(stale))
    monkeypatch.setenv("CXX", str(tmp_path / "no-compiler"))
    assert not build.build_native_or_none()
    assert not stale.exists() and "no module" in capsys.readouterr().err


def cases(device):
    """(name, function, arguments) of every call that has a native form, plain inputs."""
    g = torch.Generator().manual_seed(7)

    def bits(*shape):
        return torch.randint(-2 ** 31, 2 ** 31, shape, generator=g).to(torch.int32).to(device)

    def ternary(*shape):
        return torch.randint(-1, 2, shape, generator=g).to(torch.int8).to(device)

    def th(n):
        return torch.randint(-20, 21, (n,), generator=g).to(torch.int32).to(device)

    def randn(*shape):
        return torch.randn(shape, generator=g).to(device)

    gpu = device == "cuda"
    blob = lambda w: B.pack_weights(w) if gpu else torch.zeros(64, dtype=torch.uint8)        # noqa: E731
    tblob = lambda w: B.pack_tconv_weights(w) if gpu else torch.zeros(64, dtype=torch.uint8)  # noqa: E731
    a, low, half = bits(2, 9, 14, 2), bits(2, 9, 14, 1), bits(2, 4, 7, 4)
    even, full = bits(1, 8, 12, 2), bits(1, 4, 6, 4)
    return [
        ("conv", B.conv3x3_masked_binary, (a, 64, blob(ternary(96, 3, 3, 64)), 96, th(96))),
        ("fused, pooled", B.conv3x3_masked_binary_fused, (a, 64, None, 0, blob(ternary(64, 3, 3, 64)), 64, th(64), True, True)),
        ("fused, two", B.conv3x3_masked_binary_fused, (even, 64, full, 128, blob(ternary(64, 3, 3, 192)), 64, th(64))),
        ("concat", B.conv3x3_masked_binary_concat, (a, 64, low, 32, blob(ternary(64, 3, 3, 96)), 64, th(64), True)),
        ("two inputs", B.conv3x3_masked_binary_two_inputs, (a, 64, half, 128, True, blob(ternary(64, 3, 3, 192)), 64, th(64))),
        ("tconv", B.tconv2x2_masked_binary, (a, 64, tblob(ternary(32, 2, 2, 64)), 32, th(32))),
        ("pack float", B.pack_act, (randn(2, 5, 7, 40),)),
        ("pack int8", B.pack_act, (ternary(2, 5, 7, 64),)),
        ("stem", B.stem_fp32, (randn(1, 3, 10, 33), randn(64, 3, 3, 3))),
        ("classifier", B.classifier_fp32, (a, 64, randn(19, 64), randn(19))),
    ]


def test_the_module_has_no_thread_local_storage():
    """A library with a thread-local segment that nothing touches sends every access of torch's own
    thread-local state down the slow path of the dynamic linker for the rest of the process."""
    B.lib()
    elf = open(B.NATIVE_PATH, "rb").read()
    assert elf[:6] == b"\x7fELF\x02\x01"
    at, (size, n) = struct.unpack_from("<Q", elf, 32)[0], struct.unpack_from("<HH", elf, 54)
    kinds = [struct.unpack_from("<I", elf, at + i * size)[0] for i in range(n)]
    assert 1 in kinds and 7 not in kinds                     # PT_LOAD, PT_TLS


def flat(r):
    return list(r) if isinstance(r, tuple) else [r]


NAMES = [n for n, _, _ in cases("cpu")]


@pytest.mark.parametrize("name", NAMES)
def test_host_tensors_are_left_to_the_general_code(name):
    """... which refuses them as it does without the native calls."""
    _, f, args = next(c for c in cases("cpu") if c[0] == name)
    with pytest.raises(ValueError, match="expected a device tensor"):
        f(*args)


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_native_calls_return_what_the_general_code_returns(name, monkeypatch):
    _, f, args = next(c for c in cases("cuda") if c[0] == name)
    native = B._native()
    taken = []

    class Watch:
        def __getattr__(self, call):
            return lambda *a: taken.append(getattr(native, call)(*a)) or taken[-1]

    monkeypatch.setattr(B, "_calls", Watch())
    got = flat(f(*args))
    assert len(taken) == 1 and taken[0] is not None
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        other = flat(f(*args))
    torch.cuda.current_stream().wait_stream(side)
    monkeypatch.setattr(B, "_calls", General())
    ref = flat(f(*args))
    torch.cuda.synchronize()
    assert len(got) == len(ref) == len(other)
    for x, y, z in zip(got, ref, other):
        if y is None:
            assert x is None and z is None
            continue
        assert type(x) is type(y) and x.shape == y.shape and x.dtype == y.dtype and x.device == y.device
        assert x.is_contiguous() and not x.requires_grad
        assert torch.equal(x, y) and torch.equal(z, y)


@pytest.mark.gpu
def test_inputs_given_other_data_by_another_thread():
    """A call takes an input as it is when it checks it: pointer and sizes belong together, whatever another
    thread sets the tensor to meanwhile."""
    g = torch.Generator(device="cuda").manual_seed(11)
    small = torch.randn((1, 3, 5, 40), generator=g, device="cuda")
    large = torch.randn((2, 60, 70, 64), generator=g, device="cuda")
    expected = {r.shape: r for r in (B.pack_act(small), B.pack_act(large))}
    x, stop = torch.empty(0, device="cuda"), threading.Event()
    x.data = small

    def swap():
        for t in itertools.cycle((large, small)):
            x.data = t
            if stop.is_set():
                return

    other = threading.Thread(target=swap)
    other.start()
    try:
        got = [B.pack_act(x) for _ in range(300)]   # (the lock comes back after 5 ms)
    finally:
        stop.set()
        other.join()
    torch.cuda.synchronize()
    assert {r.shape for r in got} == set(expected)           # both were met
    for r in got:
        assert torch.equal(r, expected[r.shape])


class Sub(torch.Tensor):
    pass


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_native_calls_refuse_what_the_general_code_refuses(name, monkeypatch):
    _, f, args = next(c for c in cases("cuda") if c[0] == name)

    def outcome(a):
        """Result, or the error's type, code and message."""
        try:
            r = flat(f(*a))
        except torch.OutOfMemoryError as e:      # (its message holds the amounts in use)
            return type(e), None, None
        except (ValueError, TypeError, AttributeError, RuntimeError, ctypes.ArgumentError) as e:
            return type(e), getattr(e, "code", None), str(e)
        torch.cuda.synchronize()
        return [None if t is None else t.as_subclass(torch.Tensor).clone() for t in r]

    # (nothing that the library would take for a larger tensor than it is)
    variants = []
    for i, v in enumerate(args):
        def swap(x, i=i):
            return args[:i] + (x,) + args[i + 1:]
        if isinstance(v, torch.Tensor):
            variants += [swap(v.cpu()), swap(v.to(torch.int16)), swap(v.as_subclass(Sub)),
                         swap(torch.nn.Parameter(v) if v.is_floating_point() else v)]
            if v.dim() > 1:
                variants += [swap(v.transpose(0, -1).contiguous().transpose(0, -1))]
            if i == 0:
                variants += [swap(v[None]), swap(v.flatten()), swap(v[:0]), swap(None)]
        elif isinstance(v, int) and not isinstance(v, bool):
            variants += [swap(-v - 1), swap(2 ** 40), swap(float(v)), swap(str(v)), swap(None)]
    native = B._native()
    for a in variants:
        monkeypatch.setattr(B, "_calls", native)
        got = outcome(a)
        monkeypatch.setattr(B, "_calls", General())
        ref = outcome(a)
        assert type(got) is type(ref), (a, got, ref)
        if isinstance(ref, tuple):
            assert got == ref, a
        else:
            assert all((x is None and y is None) or torch.equal(x, y) for x, y in zip(got, ref)), a
