"""MI355X-native clustered-head decode attention (CHAI): Python face of the C-ABI library libchai.so.

The binding (and with it the shared library) is loaded on first use, so that `paper_2403_08058_amd.build` can be
imported to (re)build the library even when no library, or a stale one, is present.  There is no fallback: using
any entry point without a built library raises ImportError.
"""
import importlib

_BINDING_NAMES = ("CHAI_BF16", "CHAI_F32", "CHAI_OK", "EXPORTS", "LIB_PATH", "ChaiError", "alloc_workspace", "lib")


def __getattr__(name):
    if name == "build":
        return importlib.import_module(".build", __name__)
    binding = importlib.import_module(".binding", __name__)
    if name == "binding":
        return binding
    if name in _BINDING_NAMES or name in binding.EXPORTS:
        # Kept as an ordinary attribute until it is replaced in the binding: the next use does not come here again (an import
        # statement's worth of look-ups, 4 us per call, nearly as much as the smallest decode call takes on the GPU: 1 row x 32 fp32
        # heads, 256 tokens 10.3 -> 6.6 us).
        value = globals()[name] = getattr(binding, name)
        return value
    raise AttributeError(f"module {__name__!r} has no attribute {name!r}")
