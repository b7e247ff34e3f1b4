"""Which scan kernel serves a match call (fm_debug_scan_name), on the CPU: the
choice is made on the host from the sizes alone."""
import pytest

import paper_2502_05370_amd as fm


def test_names_follow_the_sizes():
    name = fm.debug_scan_name
    assert name(32, 8, 1000, 8) == "k_traj_split 1x1"
    assert name(24, 60, 1000000, 512, 1, "bf16") == "k_traj_mm"
    assert name(24, 60, 50000, 64) == "k_traj_scan"
    assert name(32, 16, 200000, 512, 4).startswith("k_traj_scan")
    assert name(32, 8, 1000, 8, d_emb=4096) == "k_sem_split 1x1"
    assert name(24, 60, 1000000, 512, d_emb=2048) == "k_sem_mm 256"
    assert name(32, 8, 100000, 100, d_emb=4096) == "k_sem_mm 128"
    for k in (2, 8):
        assert name(32, 8, 1000, 8, k, d_emb=4096) == "k_sem_scan"
    # both kinds on one store: max_depth says which
    assert name(32, 8, 1000, 8, d_emb=4096, max_depth=5).startswith("k_traj_")
    # the dense form has no split-depth scan
    assert name(32, 8, 1000, 8, 0) == "k_traj_scan"
    # a batch of several launches: its first one
    assert name(24, 60, 200000, 5000, 1, "bf16") == name(24, 60, 200000, 1024, 1, "bf16")


@pytest.mark.parametrize("kw", [dict(L=0), dict(L=65), dict(E=0), dict(E=65), dict(n=-1), dict(B=0), dict(B=65537), dict(k=9),
                                dict(k=-1), dict(d_emb=100), dict(max_depth=33), dict(max_depth=0)])
def test_sizes_that_no_call_takes(kw):
    a = dict(L=32, E=8, n=1000, B=8, k=1, d_emb=0)
    a.update(kw)
    with pytest.raises(ValueError, match="no match call"):
        fm.debug_scan_name(**a)


# (entries, d, queries, time of the call on k_sem_mm, on the best split-k shape), us
SEMANTIC = [(1000, 4096, 8, 92.6, 11.8), (955, 768, 8, 26.6, 8.4), (3540, 2048, 109, 53.9, 14.8), (3503, 768, 161, 28.8, 13.9),
            (46724, 1024, 1, 35.3, 21.4), (439127, 128, 29, 36.5, 74.4), (223998, 128, 33, 25.8, 56.2),
            (13308, 128, 472, 17.4, 29.4), (720906, 128, 7, 48.0, 97.0), (31848, 128, 119, 16.1, 21.0),
            (107404, 384, 38, 26.8, 34.5), (380356, 256, 12, 44.9, 59.6)]


@pytest.mark.parametrize("n,d,B,mm,split", SEMANTIC)
def test_semantic_search_takes_the_scan_that_measured_faster(n, d, B, mm, split):
    assert fm.debug_scan_name(32, 8, n, B, d_emb=d).startswith("k_sem_mm" if mm < split else "k_sem_split")


# (L, E, maps, queries, matches, type, time of the call on the other trajectory
# scan, on the best split-depth shape), us
TRAJECTORY = [(32, 8, 1000, 8, 1, "f32", 18.6, 14.3), (61, 33, 320, 2, 1, "f32", 64.1, 14.9),
              (48, 32, 272, 281, 1, "f32", 79.3, 27.1), (24, 60, 6766, 4, 1, "f32", 36.3, 15.6),
              (61, 33, 1699, 10, 1, "bf16", 52.7, 20.6), (61, 33, 28275, 2, 1, "bf16", 52.0, 23.5),
              (7, 4, 7223, 234, 4, "bf16", 39.8, 24.0),
              (24, 60, 72606, 130, 1, "f32", 129.1, 339.8), (24, 64, 53410, 79, 1, "f32", 83.0, 201.7),
              (24, 60, 23877, 322, 1, "f32", 98.8, 182.8), (26, 60, 20420, 80, 1, "f32", 48.7, 72.8),
              (26, 60, 8994, 451, 1, "f32", 60.4, 120.4), (48, 32, 39534, 191, 1, "bf16", 44.0, 82.8),
              (48, 32, 21317, 541, 1, "f32", 129.6, 215.3), (24, 64, 18824, 160, 1, "f32", 48.5, 84.4),
              (16, 20, 79793, 870, 8, "f32", 323.0, 569.0), (32, 16, 79793, 870, 8, "f32", 342.0, 574.0)]


@pytest.mark.parametrize("L,E,n,B,k,dtype,other,split", TRAJECTORY)
def test_trajectory_search_takes_the_scan_that_measured_faster(L, E, n, B, k, dtype, other, split):
    assert fm.debug_scan_name(L, E, n, B, k, dtype).startswith("k_traj_split") == (split < other)


# (L, E, maps, queries, matches, type, time of the call with ranking floors, without), us
FLOORS = [(32, 16, 84064, 689, 1, "f32", 148.4, 160.9), (12, 12, 56666, 695, 8, "f32", 237.3, 261.2),
          (32, 8, 187879, 306, 8, "f32", 213.9, 262.5), (24, 60, 62658, 1007, 1, "f32", 266.0, 327.1),
          (24, 60, 102912, 433, 8, "bf16", 243.6, 251.5), (12, 40, 163634, 793, 8, "bf16", 426.2, 583.6),
          (32, 8, 30452, 142, 1, "f32", 30.6, 29.1), (12, 12, 112923, 127, 8, "bf16", 97.5, 89.8),
          (24, 60, 40658, 205, 1, "f32", 84.9, 78.8), (16, 20, 91654, 44, 8, "f32", 76.7, 70.7),
          (24, 60, 34393, 512, 1, "f32", 126.7, 118.3), (32, 8, 46879, 160, 8, "bf16", 74.3, 67.3),
          (1, 16, 56892, 428, 1, "bf16", 31.1, 37.4), (2, 8, 100741, 144, 1, "f32", 34.3, 40.3),
          (2, 8, 32409, 167, 1, "bf16", 25.8, 23.6)]


@pytest.mark.parametrize("L,E,n,B,k,dtype,with_floors,without", FLOORS)
def test_ranking_floors_serve_the_launches_that_measured_faster(L, E, n, B, k, dtype, with_floors, without):
    assert fm.debug_scan_name(L, E, n, B, k, dtype) == ("k_traj_scan floors" if with_floors < without else "k_traj_scan")


# the sizes of the GPU test of the floors that reach them
@pytest.mark.parametrize("dtype,E,k,B,n", [("f32", 16, 4, 1000, 33001), ("f32", 8, 8, 600, 20011), ("f32", 60, 1, 600, 60003),
                                           ("bf16", 60, 8, 1000, 40003), ("bf16", 16, 3, 1000, 40007)])
def test_floor_test_reaches_the_floors(dtype, E, k, B, n):
    assert fm.debug_scan_name(5, E, n, B, k, dtype) == "k_traj_scan floors"


# (L, E, maps, queries, time of the call on k_traj_scan, on k_traj_mm), us: bf16,
# one match, half a band of k_traj_mm
HALF_BAND = [(32, 16, 105953, 109, 42.6, 39.1), (32, 8, 185776, 114, 45.9, 41.5), (32, 8, 293509, 115, 64.9, 56.0),
             (16, 20, 145156, 119, 57.7, 48.5), (24, 60, 215644, 97, 147.7, 127.1), (24, 64, 309628, 114, 201.4, 197.7),
             (24, 60, 195589, 107, 144.6, 108.9), (24, 64, 127247, 126, 113.2, 93.9), (24, 64, 193368, 118, 152.6, 128.5),
             (24, 60, 111618, 123, 82.6, 87.4), (24, 60, 159606, 113, 116.1, 120.4), (24, 64, 122243, 112, 88.3, 91.4)]


@pytest.mark.parametrize("L,E,n,B,scan,mm", HALF_BAND)
def test_half_a_band_takes_the_scan_that_measured_faster(L, E, n, B, scan, mm):
    assert fm.debug_scan_name(L, E, n, B, 1, "bf16") == ("k_traj_mm" if mm < scan else "k_traj_scan")


# the sizes of the GPU tests of the split scans, and the shapes that they reach
@pytest.mark.parametrize("shape,n,d,B", [("1x1", 250, 4096, 17), ("4x1", 4100, 2048, 8), ("4x2", 1052, 4096, 450),
                                         ("4x4", 4100, 640, 129), ("4x8", 12007, 2048, 100)])
def test_semantic_split_test_reaches_every_shape(shape, n, d, B):
    assert fm.debug_scan_name(2, 4, n, B, d_emb=d) == f"k_sem_split {shape}"


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape,E,L,n,B", [("1x1", 60, 24, 1003, 33), ("2x2", 60, 6, 4100, 200), ("2x4", 8, 32, 4100, 100)])
@pytest.mark.parametrize("k", [1, 3, 8])
def test_trajectory_split_test_reaches_every_shape(shape, E, L, n, B, k, dtype):
    assert fm.debug_scan_name(L, E, n, B, k, dtype) == f"k_traj_split {shape}"
