"""Default sweep workgroup sizes against measured sweep times (us, ten sweeps of
a launch on MI355X; lanes: time), columns few and many.  A shape where two
columns just fit a CU's LDS with a small workgroup took that size, at up to
twice the time of a large one."""
import ctypes
import os

import pytest

#         d, L, glass, columns: times by lanes
MEASURED = {
    (2, 96, False, 313): {128: 799, 192: 769, 256: 613, 320: 658, 384: 547, 448: 496, 512: 441, 576: 489, 640: 478,
                          704: 436, 768: 395},
    (3, 20, True, 400): {128: 804, 192: 756, 256: 596, 320: 646, 384: 561, 448: 492, 512: 441, 576: 504, 640: 478,
                         704: 432, 768: 414},
    (2, 88, True, 257): {64: 954, 128: 667, 192: 460, 256: 535, 320: 567, 384: 488, 448: 425, 512: 386, 576: 430,
                         640: 419, 704: 364, 768: 360},
    (2, 32, False, 313): {64: 140, 128: 106, 192: 86, 256: 71, 320: 77, 384: 88, 448: 81, 512: 76, 576: 95, 640: 95,
                          704: 94, 768: 95},
    (3, 16, True, 313): {64: 595, 128: 421, 192: 299, 256: 217, 320: 263, 384: 262, 448: 226, 512: 196, 576: 287,
                         640: 278, 704: 258, 768: 223},
    (2, 16, False, 1): {64: 46, 128: 35, 192: 35, 256: 35, 320: 35, 384: 36, 448: 36, 512: 37, 576: 36, 640: 37,
                        704: 37, 768: 40},
    (3, 10, True, 512): {64: 166, 128: 124, 192: 98, 256: 81, 320: 86, 384: 98, 448: 91, 512: 86, 576: 106, 640: 106,
                         704: 107, 768: 106},
    (2, 32, False, 3100): {64: 336, 128: 295, 192: 333, 256: 315, 320: 466, 384: 496, 448: 467, 512: 421, 576: 568,
                           640: 567, 704: 572, 768: 583},
    (2, 30, True, 3100): {64: 338, 128: 300, 192: 336, 256: 313, 320: 475, 384: 495, 448: 466, 512: 423, 576: 564,
                          640: 568, 704: 567, 768: 569},
    (3, 8, True, 5000): {64: 249, 128: 276, 192: 357, 256: 347, 320: 522, 384: 522, 448: 497, 512: 477, 576: 743,
                         640: 754, 704: 770, 768: 772},
    (2, 28, False, 5000): {64: 364, 128: 391, 192: 456, 256: 445, 320: 720, 384: 714, 448: 647, 512: 618, 576: 861,
                           640: 866, 704: 872, 768: 875},
    (2, 64, False, 1600): {64: 1165, 128: 812, 192: 703, 256: 553, 320: 819, 384: 742, 448: 627, 512: 564, 576: 845,
                           640: 832, 704: 776, 768: 714},
    (3, 12, True, 4200): {64: 979, 128: 830, 192: 763, 256: 699, 320: 1014, 384: 1047, 448: 935, 512: 866, 576: 1223,
                          640: 1218, 704: 1228, 768: 1218},
    (2, 128, False, 1000): {192: 2885, 256: 2059, 320: 2268, 384: 1884, 448: 1704, 512: 1444, 576: 1744},
}


@pytest.mark.parametrize("shape", sorted(MEASURED))
def test_size_is_near_the_fastest(shape):
    from paper_2401_07965_amd import build, pa
    if not os.path.exists(pa.LIB_PATH):
        build.build()
    f = ctypes.CDLL(pa.LIB_PATH)["_Z24pa_default_sweep_threadsiibl"]
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int64], ctypes.c_int
    d, L, glass, columns = shape
    times = MEASURED[shape]
    lanes = f(L ** d, d, glass, columns)
    # what the rule keeps to on 95 of 100 measured shapes of ten sweeps
    assert lanes in times and times[lanes] <= 1.08 * min(times.values()), (lanes, times)


@pytest.mark.gpu
def test_batches_and_runs_take_it():
    """The size a batch reports for a shape that two small workgroups a CU would just hold."""
    from paper_2401_07965_amd import pa
    b = pa.PABatch([dict(dim=2, L=96, R=64 * 300)], max_points=2)
    assert b.groups()[0] >= 512
    b.close()
