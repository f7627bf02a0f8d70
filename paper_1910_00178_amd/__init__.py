"""MI355X (gfx950) u8 x s8 -> s32 GEMM: thin binding over the C-ABI HIP library.

The binding (and with it the shared library) is loaded on first use of any of its names, so
that `paper_1910_00178_amd.build` can (re)compile the library without loading a stale one.
There is no fallback: a missing or unloadable library raises.
"""
import importlib
import types

_binding = None
_found = set()           # names of the binding that this module holds as well


class _Binding(types.ModuleType):
    """The binding's module: a name that is set or deleted there is looked up again here, all of them after a reload."""

    def __setattr__(self, name, value):
        super().__setattr__(name, value)
        for n in list(_found) if name == "__spec__" else [name]:       # a reload begins by setting it
            _forget(n)

    def __delattr__(self, name):
        super().__delattr__(name)
        _forget(name)


def _forget(name):
    if name in _found:
        _found.discard(name)
        globals().pop(name, None)


def _load():
    global _binding
    if _binding is None:
        _binding = importlib.import_module(".binding", __name__)
        _binding.__class__ = _Binding
    return _binding


def __getattr__(name):
    if name.startswith("__"):
        raise AttributeError(name)
    if name in ("build", "workloads", "binding"):
        return importlib.import_module("." + name, __name__)
    value = getattr(_load(), name)
    if not name.startswith("_"):
        globals()[name] = value      # found without this function from now on (it costs 0.2 us a call)
        _found.add(name)
    return value


def __dir__():
    return sorted(set(globals()) | set(dir(_load())))
