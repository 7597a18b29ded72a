"""The backward launcher refuses arguments that contradict themselves, before
anything is launched (CPU)."""
import host_groups as hg

HIP_ERROR_INVALID_VALUE = 1


def test_group_partials_without_streamed_rows_are_refused():
    """The plan sizes the partial gradients by sibling groups exactly where the
    bf16 query pass streams.  A slice past the 32-bit token range does not
    stream: its per-block partial rows would not fit the groups' space."""
    import ctypes
    fn = hg.library().host_backward_status
    fn.argtypes = [ctypes.c_int64, ctypes.c_int]
    assert fn(2 ** 31 - 64, 1 << 20) == HIP_ERROR_INVALID_VALUE
