"""Which 3x3 weight gradients take all nine taps in one workgroup, in how many slices: the library's rule (no GPU)."""
import ctypes as C

import paper_2111_10672_amd as spb

# (images, size, channels), us as a gathering product, us here
TIMED = [
    ((48, 13, 128), 14.2, 16.0), ((24, 13, 128), 12.1, 14.7), ((48, 8, 128), 11.8, 14.9), ((24, 7, 256), 11.7, 14.7), ((48, 4, 256), 10.0, 14.6),
    ((24, 8, 256), 12.4, 15.7), ((24, 4, 512), 12.6, 17.6),
    ((128, 32, 64), 50, 25), ((128, 16, 128), 32, 25), ((128, 8, 256), 29, 27), ((128, 4, 512), 33, 30), ((48, 49, 64), 44.4, 26.2), ((96, 32, 64), 37.6, 24.1),
]


def splits(shapes):
    """What the library answers: the layout of ConvGeom is n, sh, sw, sc, rh, rw, r, s, stride, pad, pad_w, transposed, w_cin, w_cout."""
    ask = getattr(spb.lib(), "_ZN3spb18conv3_wgrad_splitsERKNS_8ConvGeomEi")
    ask.restype, ask.argtypes = C.c_int, [C.c_void_p, C.c_int]
    return [ask(C.byref((C.c_int * 14)(n, i, i, cin, i, i, 3, 3, 1, 1, 1, 0, 0, 0)), cout) for n, i, cin, cout in shapes]


def test_each_timed_shape_goes_to_the_faster_kernel():
    got = splits([(n, i, c, c) for (n, i, c), _, _ in TIMED])
    wrong = [t for t, s in zip(TIMED, got) if (s > 0) != (t[2] < t[1])]
    assert len(got) == len(TIMED) and not wrong, wrong


def test_slices_follow_the_workgroups():
    # one block of channels, four, 64; long ranges of pixels take half as many more, however long
    assert splits([(128, 32, 64, 64), (128, 16, 128, 128), (128, 4, 512, 512)]) == [128, 32, 2]
    assert splits([(256, 64, 64, 64), (2560, 64, 64, 64), (256, 64, 128, 128), (48, 13, 512, 512)]) == [192, 192, 48, 3]
    # channels that are not whole 64-groups
    assert splits([(128, 32, 96, 96)]) == [0]
