"""A network is made and destroyed without a GPU (its calls need one), as its sizes are asked for."""
import ctypes


def test_create_and_destroy_without_a_device():
    from paper_2408_14778_amd import _native as N
    lib = N.load()
    F, H, A, batch = 96, 64, 4, 32
    need = lib.cfr_mlp_workspace_bytes(F, H, A, batch)
    ws = ctypes.create_string_buffer(need)  # never read or written by these calls
    h = ctypes.c_void_p()
    rc = lib.cfr_mlp_create(F, H, A, batch, ctypes.cast(ws, ctypes.c_void_p), ctypes.c_size_t(need), None,
                            ctypes.byref(h))
    assert rc == 0 and h.value
    assert lib.cfr_mlp_destroy(h) == 0
    h = ctypes.c_void_p()
    rc = lib.cfr_mlp_create(F, H, A, batch, ctypes.cast(ws, ctypes.c_void_p), ctypes.c_size_t(1), None,
                            ctypes.byref(h))
    assert N.ERRORS[rc] == "CFR_ENOMEM"
