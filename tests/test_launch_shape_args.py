"""scps_get_launch_shape checks its arguments on the host."""
import ctypes as C


def test_null_arguments_are_refused():
    from paper_1705_02180_amd import scps
    out = (C.c_int32 * 3)()
    assert scps._lib.scps_get_launch_shape(None, None) == -1
    assert scps._lib.scps_get_launch_shape(None, C.cast(out, C.c_void_p)) == -1
    assert scps.KERNELS[1] == "persistent" and len(scps.KERNELS) == 5
