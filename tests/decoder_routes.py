"""Sizes for the planar decoder's kernels: where the limits between them move, test_host_calls.py fails for the sizes here
that no longer take the kernel they are meant for."""
MB = 1 << 20
ROUTES = ("direct4", "direct8", "scan4", "scan8", "scan4 large", "two")


def elements(route, w, first=0, dense=False):
    """A size whose output, from element `first` of an aligned buffer on, is written by workgroups of 4 or 8 waves that
    count for themselves (direct) or scan, or by two launches.  dense: three quarters of the elements or more are stored."""
    two = 45 if first * w % 16 == 0 else 77 if dense else 57
    return {"direct4": 5 * (4096 // w) + 3, "direct8": 60 * 8192 + 3, "scan4": 3 * MB // w + 3, "scan8": 17 * MB // w + 3,
            "scan4 large": 36 * MB // w + 3, "two": two * MB // w + 3}[route]
