"""Which kernel a run takes, and runs held to the stage kernels (test hooks of
the library that are not part of its ABI)."""

import contextlib
import ctypes


def _lib():
    import paper_1803_03498_amd as heom
    lib = heom.load()
    lib.heom_test_run_kernel.argtypes = [ctypes.c_void_p, ctypes.c_int32]
    lib.heom_test_run_kernel.restype = ctypes.c_char_p
    for name in ("heom_test_packed_min", "heom_test_columns_min"):
        getattr(lib, name).argtypes = [ctypes.c_int64]
        getattr(lib, name).restype = None
    lib.heom_test_resident_off.argtypes = [ctypes.c_int32]
    lib.heom_test_resident_off.restype = None
    return lib


def run_kernel(prob, precision, herm=True):
    """The kernel of the ADOs u >= 1 in a run on this thread."""
    import paper_1803_03498_amd as heom
    p = heom.Problem(prob, precision)
    name = _lib().heom_test_run_kernel(ctypes.byref(p.struct), 1 if herm else 0)
    assert name is not None
    return name.decode()


@contextlib.contextmanager
def forms(resident=True, packed_min=-1, columns_min=-1):
    """This thread's runs without the resident form, packed from packed_min
    elements and in tiles from columns_min of them on (-1: as the library does)."""
    lib = _lib()
    lib.heom_test_resident_off(0 if resident else 1)
    lib.heom_test_packed_min(packed_min)
    lib.heom_test_columns_min(columns_min)
    try:
        yield
    finally:
        lib.heom_test_resident_off(0)
        lib.heom_test_packed_min(-1)
        lib.heom_test_columns_min(-1)


def stages_only():
    return forms(resident=False, packed_min=1 << 62, columns_min=1 << 62)
