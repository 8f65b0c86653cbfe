"""The native argument marshalling against the binding's own Python functions: the same results, and the same exceptions,
for every form of argument that either takes."""
import sys

import numpy as np
import pytest
import torch

from paper_2302_02390_amd import binding as qb
from gpu_util import DEV, synth

pytestmark = pytest.mark.gpu

N, B = 3 * 1024 + 40, 1024


def _call(name, *args):
    """(exception type, message) of the native function and of the Python one, None for a plain return."""
    qb.lib()
    got = []
    for f in (getattr(qb, name), qb._IN_PYTHON[name]):
        try:
            f(*args)
            got.append(None)
        except Exception as e:
            got.append((type(e), str(e)))
    return got


def _step(launch, **changed):
    x, g = (torch.from_numpy(a).to(DEV) for a in synth(N, 3))
    codes, meta = qb.alloc_packed(N, 8, B, DEV)
    sat = torch.zeros(1, dtype=torch.int64, device=DEV)
    a = dict(x=x, g=g, n=N, lr=1e-3, wbits=8, gbits=4, bucket=B, delta=0.0, seed=5, offset=0, codes=codes,
             meta=meta.reshape(-1), sat=sat)
    a.update({k: v(a) if callable(v) else v for k, v in changed.items()})
    try:
        launch(x, "qsdp_fused_step", *a.values())
    except Exception as e:
        return type(e), str(e)
    return [t.cpu() for t in (x, codes, meta, sat)]


@pytest.mark.parametrize("changed", [
    dict(), dict(seed=-1), dict(seed=2 ** 64 + 7), dict(seed=np.int64(9)), dict(seed=True), dict(n=np.int32(N)),
    dict(lr=1), dict(lr=np.float32(1e-3)), dict(lr=np.float64(1e-3)), dict(lr=lambda a: torch.tensor(1e-3)),
    dict(lr=lambda a: torch.tensor(1e-3, device=DEV)), dict(n=lambda a: torch.tensor(N)), dict(sat=None),
    dict(codes=None, meta=None), dict(x=lambda a: a["x"].data_ptr()), dict(x=lambda a: torch.nn.Parameter(a["x"])),
    dict(wbits=9), dict(offset=3), dict(x=lambda a: a["x"][1:]), dict(lr="1"), dict(seed=1.5), dict(seed="1"),
    dict(n=None), dict(lr=10 ** 400), dict(x=None), dict(codes=1.5)])
def test_arguments_of_a_launch(changed):
    qb.lib()
    native, python = _step(qb._launch, **changed), _step(qb._IN_PYTHON["_launch"], **changed)
    if isinstance(python, tuple):
        assert native == python
    else:
        assert all(torch.equal(a, b) for a, b in zip(native, python))


def test_arguments_too_few_too_many_and_names():
    x = torch.zeros(64, device=DEV)
    for args in ((), (x,), (x, "qsdp_fused_step"), (x, "qsdp_fused_step", x), (x, "nothing_of_the_kind", x),
                 (x.cpu(), "qsdp_fit_levels", x, 64, 4, 32, 0.1, 0, x), (None, "qsdp_fused_step"), (x, 3),
                 (x, "qsdp_fit_levels", x, 64, 4, 32, 0.1, 0, x, None, None)):
        native, python = _call("_launch", *args)
        assert native == python, args
    lv = qb.levels_uniform(4, DEV)
    assert _call("_launch", x, "".join(["qsdp_", "fit_levels"]), x, 64, 4, 32, 0.1, 0, lv) == [None, None]


def test_checks():
    x = torch.zeros((6, 64), device=DEV)
    ints, longs = x.to(torch.int32), x.to(torch.int64)
    fits = lambda *a: (_call("_packed_ok", *a), _call("_rows_ok", *a))
    for t in (x, x.t(), x[:, ::2], x[:, :32], x[:1, :1], x.half(), x.cpu(), torch.nn.Parameter(x), x.to_sparse(), None, 3,
              np.zeros((2, 2), np.float32)):
        for name in ("_is", "_is_rows"):
            native, python = _call(name, t, torch.float32)
            assert native == python, (name, t)
    for outputs in ((None, None, None), (ints, x, longs), (ints, None, None), (x, x, longs), (ints, x, ints),
                    (ints.cpu(), x, None), (None, x.t(), None), (None, None, 3)):
        native, python = _call("_step_outputs", *outputs)
        assert native == python, outputs
    for codes, meta in ((ints, x), (ints, None), (None, x), (None, None), (x, ints)):
        for n in (0, 1, 64, 65, 256, 384, 385, 1 << 40, -5, np.int64(64)):
            for bits, bucket in ((8, 32), (4, 1024), (9, 32), (8, 33), (0, 32)):
                for native, python in fits(codes, meta, n, bits, bucket):
                    assert native == python, (codes is None, meta is None, n, bits, bucket)


def test_tensors_on_one_device():
    gpu, cpu = torch.zeros(64, device=DEV), torch.zeros(64)
    segs = qb.Segments([64], 32, DEV)
    elsewhere = qb.Segments([64], 32, "cpu")
    for args in ((), (gpu,), (cpu,), (gpu, gpu), (gpu, cpu), (cpu, gpu), (cpu, cpu), (gpu, 3, 1.5, None, True, gpu),
                 (gpu, 3, cpu), (gpu, np.float32(1), gpu), (gpu, np.float32(1), cpu), (gpu, torch.nn.Parameter(gpu)),
                 (gpu, torch.nn.Parameter(cpu)), (gpu, segs), (gpu, elsewhere), (cpu, segs), (gpu, (gpu, 1)),
                 (gpu, [gpu, cpu]), (gpu, (cpu, 1.0)), (gpu, "cpu"), (gpu, torch.device("cpu")), (gpu, [])):
        for kwargs in ({}, {"a": 1, "b": gpu}, {"a": cpu}, {"a": None, "segs": segs}, {"adamw": (gpu, cpu)}):
            native, python = _call("_devices_ok", "an entry point", args, kwargs)
            assert native == python, (args, kwargs)
    with pytest.raises(ValueError, match="qsdp_quantize_grad: tensors on cuda:0 and on cpu"):
        qb.qsdp_quantize_grad(gpu, 4, 32, 1, 0, cpu.to(torch.int32), cpu)
    for args in ((), ("name",), ("name", [gpu, cpu], {}), ("name", (gpu, cpu), None), (1, 2, 3)):
        native, python = _call("_devices_ok", *args)
        assert native == python or native[0] is python[0], args


def test_segment_tables_on_one_device():
    """A table's own tensor decides, also where it has none, another object, or a subclass of the table's type."""
    gpu, cpu = torch.zeros(64, device=DEV), torch.zeros(64)

    class Special(qb.Segments):
        pass

    tables = {"gpu": qb.Segments([64], 32, DEV), "cpu": qb.Segments([64], 32, "cpu"), "special": Special([64], 32, DEV),
              "special cpu": Special([64], 32, "cpu")}
    for name, value in (("none", None), ("text", "cpu"), ("parameter", torch.nn.Parameter(gpu)), ("missing", ...)):
        tables[name] = qb.Segments([64], 32, DEV)
        if value is ...:
            del tables[name].device
        else:
            tables[name].device = value
    for name, t in tables.items():
        held = t.__dict__.get("device")
        before = sys.getrefcount(held)
        for args in ((t,), (gpu, t), (t, gpu), (cpu, t), (t, cpu), (gpu, t, 3, t), (t, tables["gpu"]), (tables["cpu"], t)):
            for kwargs in ({}, {"segs": t}, {"segs": t, "x": gpu}, {"x": cpu}):
                native, python = _call("_devices_ok", "an entry point", args, kwargs)
                assert native == python, (name, len(args), sorted(kwargs))
        assert held is None or sys.getrefcount(held) == before, name


def test_segment_tables_are_looked_at_in_native_code():
    gpu, segs = torch.zeros(64, device=DEV), qb.Segments([64], 32, DEV)
    qb.lib()
    native = qb._native_marshalling()
    assert native is not None
    in_python = list(qb._IN_PYTHON.values())

    def not_called(*args):
        raise AssertionError("left to Python")

    native.attach(vars(qb), *in_python[:-1], not_called)
    try:
        assert qb._devices_ok("an entry point", (gpu, segs, 4, None), {"segs": segs}) is None
        with pytest.raises(AssertionError, match="left to Python"):
            qb._devices_ok("an entry point", (gpu, qb.Segments([64], 32, "cpu")), {})
    finally:
        native.attach(vars(qb), *in_python)
