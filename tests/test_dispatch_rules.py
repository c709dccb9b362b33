"""The dispatch rules choose the faster side where both sides were measured
(forward on one MI355X, us; CPU: the rules alone, compiled for the host)."""
import pytest

from paper_2609_36070_amd.workloads import Workload
from tests import dispatch

pytestmark = pytest.mark.skipif(not dispatch.HAVE_CXX, reason="needs a host compiler")


@pytest.mark.parametrize("T,d,E,f,fs,folded,parts", [
    # d, f, experts and a shared expert in the range; both ends of each
    (100, 256, 16, 2048, 0, 670, 42), (8192, 256, 16, 2048, 0, 1194, 636), (30000, 256, 2, 256, 0, 48.6, 70.6),
    (32768, 256, 8, 256, 0, 171, 257), (4099, 256, 8, 256, 0, 78.9, 49.4), (16384, 512, 8, 256, 0, 140, 222),
    (8192, 1024, 8, 256, 0, 125, 203), (2048, 1024, 8, 1024, 0, 253, 128), (8192, 1024, 8, 1024, 0, 450, 481),
    (4000, 2048, 2, 256, 0, 42.3, 62.2), (500, 2048, 8, 768, 0, 196, 87.5), (4000, 2048, 8, 768, 0, 321, 372),
    (500, 2048, 16, 768, 1024, 405, 155), (4000, 2048, 16, 768, 1024, 706, 848), (2800, 2816, 2, 256, 512, 85, 131),
    (1536, 4096, 8, 256, 0, 140, 205), (512, 4096, 16, 2048, 0, 988, 430), (1000, 7168, 2, 256, 0, 76, 91),
    (200, 7168, 8, 2048, 2048, 706, 387), (500, 7168, 4, 2048, 2048, 493, 355),
    # one expert, and a shared expert longer than the others
    (1, 2048, 1, 1536, 0, 55.1, 38.7), (300, 256, 1, 2048, 0, 61.7, 33.8), (16000, 256, 1, 2048, 0, 138, 122),
    (16000, 256, 1, 256, 0, 29, 42.8), (2000, 1024, 1, 512, 0, 33.6, 32.2), (4000, 1024, 1, 512, 0, 36.2, 40.0),
    (1000, 4096, 1, 512, 0, 55.5, 58.6), (1000, 4096, 1, 2048, 0, 94.1, 80.0), (2000, 4096, 1, 2048, 0, 142, 154),
    (1000, 7168, 1, 2048, 2048, 208, 234), (300, 7168, 1, 2048, 1024, 195, 170), (4000, 1024, 1, 512, 1024, 87.4, 89.1),
    (2000, 1024, 1, 512, 1024, 71.6, 63.8), (4000, 256, 2, 256, 1024, 66.1, 56.3), (16000, 256, 2, 256, 1024, 112.7, 119.3),
    (2000, 1024, 2, 512, 1024, 85.4, 69.9), (4000, 1024, 3, 512, 1024, 128.3, 123.2), (1000, 4096, 3, 512, 0, 82.0, 78.2),
    (2000, 4096, 3, 512, 1024, 192.4, 239.7),
])
def test_dense_down_products(T, d, E, f, fs, folded, parts):
    w = Workload("dense", T=T, d=d, E=E, k=E, f=f, f_s=fs)
    assert dispatch.dense_parts(w) == (parts < folded)


@pytest.mark.parametrize("T,d,E,k,f,fs,small,tiles", [
    # ordinary loads (router bias of std 0.5 or a hot expert), without and with a shared expert, then top 1 and top 2 of many
    (512, 2048, 128, 8, 768, 0, 276, 333), (1000, 2048, 128, 8, 768, 0, 330, 353), (250, 4096, 32, 8, 1536, 0, 336, 341),
    (512, 3072, 16, 2, 1024, 0, 108, 117), (256, 4096, 8, 2, 2048, 0, 141, 152),
    (64, 4096, 32, 8, 1536, 2048, 284, 398), (128, 4096, 32, 8, 1536, 2048, 297, 409),
    (1000, 4096, 32, 1, 1536, 2048, 387, 418), (2000, 4096, 32, 1, 1536, 2048, 512, 506),
    (4000, 2048, 200, 1, 768, 2048, 506, 615), (8000, 2048, 200, 1, 768, 2048, 745, 739),
    (12800, 2048, 200, 1, 768, 2048, 1003, 892), (8000, 2048, 200, 1, 768, 1024, 616, 649),
    (12800, 2048, 200, 1, 768, 1024, 784, 756), (2000, 2048, 128, 2, 768, 1024, 313, 375),
])
def test_small_batches(T, d, E, k, f, fs, small, tiles):
    w = Workload("small", T=T, d=d, E=E, k=k, f=f, f_s=fs)
    assert bool(dispatch.small_tiles(w)) == (small < tiles)


def test_small_batches_bounds():
    w = Workload("small", T=128, d=256, E=4, k=2, f=512)
    assert dispatch.small_tiles(w) == 4 and dispatch.small_tiles(w.scaled(T=129)) == 0      # 64 rows per expert
    assert dispatch.small_tiles(w.scaled(T=16)) == 1 and dispatch.small_tiles(w.scaled(T=17)) == 4
    assert dispatch.small_tiles(w.scaled(T=0)) == 0
    dense = w.scaled(k=4)
    assert dispatch.small_tiles(dense.scaled(T=64)) == 4 and dispatch.small_tiles(dense.scaled(T=65)) == 0
    shared = Workload("shared", T=1024, d=256, E=64, k=1, f=256, f_s=1024)                   # T f_s = 64 E f
    assert dispatch.small_tiles(shared) == 4 and dispatch.small_tiles(shared.scaled(T=1025)) == 0
    wide = shared.scaled(f_s=32768)                                                          # one pass over its weights
    assert dispatch.small_tiles(wide.scaled(T=64)) == 4 and dispatch.small_tiles(wide.scaled(T=65)) == 0


@pytest.mark.parametrize("T,d,E,k,f,fs,us", [
    # us with 1, 2 (and 4) slices; batches whose tokens reach other experts each time
    (1, 2048, 128, 8, 768, 0, (32.5, 30.2)), (2, 2048, 128, 8, 768, 0, (37.9, 41.6)), (6, 2048, 128, 8, 768, 0, (74, 78.6)),
    (2, 4096, 32, 8, 1536, 0, (125.5, 117)), (3, 4096, 32, 8, 1536, 0, (139, 144)),
    (1, 7168, 8, 8, 2048, 2048, (186, 169, 160)), (61, 7168, 8, 8, 2048, 2048, (242, 214, 206)),
    (24, 2048, 8, 2, 1024, 0, (40.5, 36.9)), (61, 2048, 8, 2, 1024, 0, (44.1, 45.6)),
    (1, 4096, 8, 2, 2048, 0, (56, 45, 41)), (2, 4096, 8, 2, 2048, 0, (60, 50, 52)), (3, 4096, 8, 2, 2048, 0, (62, 65, 56)),
    (4, 4096, 8, 2, 2048, 0, (70, 82, 76)), (24, 4096, 8, 2, 2048, 0, (88, 92, 94)), (61, 4096, 8, 2, 2048, 0, (93, 96, 101)),
    (8, 7168, 64, 8, 512, 512, (186, 175)), (16, 7168, 64, 8, 512, 512, (230, 234)),
    (2, 5120, 200, 2, 512, 0, (56, 40, 33)), (24, 5120, 200, 2, 512, 0, (138, 129)),
    (16, 3072, 8, 2, 2048, 0, (65.8, 70)), (28, 6144, 24, 8, 1536, 1024, (326, 315)),
    (51, 4864, 8, 4, 2048, 0, (132, 141)), (4, 2048, 16, 16, 1024, 1024, (65.7, 63)),
])
def test_small_batch_slices(T, d, E, k, f, fs, us):
    w = Workload("small", T=T, d=d, E=E, k=k, f=f, f_s=fs)
    assert dispatch.kslices(w) == 2 ** us.index(min(us))


def test_small_batch_slices_bounds():
    w = Workload("small", T=1, d=2048, E=8, k=1, f=256)
    assert dispatch.kslices(w) == 2 and dispatch.kslices(w.scaled(d=4096)) == 4
    assert dispatch.kslices(w.scaled(d=1792)) == 1 and dispatch.kslices(w.scaled(d=3840)) == 2   # 1024 rows per slice
    one = Workload("one", T=1, d=2048, E=1, k=1, f=256)
    assert dispatch.kslices(one.scaled(f=64 * 128)) == 2      # 128 workgroups: one round of slices
    assert dispatch.kslices(one.scaled(f=64 * 132)) == 1      # two rounds of slices
    assert dispatch.kslices(one.scaled(f=64 * 260)) == 2      # two rounds, three of slices
    assert dispatch.kslices(one.scaled(f=64 * 516)) == 2      # three rounds, five of slices
    assert dispatch.kslices(one.scaled(f=64 * 640)) == 1
    for f, slices in ((64 * 288, 4), (64 * 320, 2), (64 * 344, 2), (64 * 388, 1)):    # as many rounds at two and at four
        assert dispatch.kslices(one.scaled(d=4096, f=f)) == slices


def test_dense_down_products_bounds():
    """Never for sparse routing, no tokens, or more tiles of Y than half of the CUs."""
    dense = Workload("dense", T=200, d=7168, E=8, k=8, f=2048, f_s=2048)
    assert dispatch.dense_parts(dense)
    assert not dispatch.dense_parts(dense.scaled(k=7))
    assert not dispatch.dense_parts(dense.scaled(T=0))
    assert dispatch.dense_parts(dense.scaled(T=1024)) and not dispatch.dense_parts(dense.scaled(T=1025))


@pytest.mark.parametrize("T,d,E,k,direct,others", [
    (1, 4096, 16, 8, 8, 12), (2048, 16384, 16, 8, 27, 37), (1, 16384, 64, 8, 37, 74), (2048, 7168, 64, 8, 26, 43),
    (2048, 4608, 128, 8, 20.2, 25.1), (500, 5120, 128, 16, 26.6, 33.0), (1024, 5120, 128, 8, 21.4, 24.2),
    (16, 5120, 128, 1, 16.6, 15.4), (16, 6144, 96, 8, 22.8, 20.6), (2048, 7168, 128, 8, 29.2, 26.3),
    (1, 8192, 160, 8, 38.2, 33.8), (16, 4608, 160, 2, 25.5, 24.2), (1024, 5120, 200, 8, 34.2, 41.2),
    (2048, 4608, 200, 8, 37.7, 41.7), (2048, 4608, 200, 2, 33.4, 31.4), (739, 7168, 200, 1, 46.9, 31.7),
    (2048, 3584, 256, 1, 27.6, 29.1), (2048, 4096, 256, 1, 31.6, 29.5), (2048, 4608, 256, 1, 35.5, 29.6),
    (16, 4096, 256, 4, 24.9, 25.1), (1024, 5120, 256, 8, 40.2, 41.6), (2048, 5120, 256, 8, 44.7, 41.7), (1600, 5120, 160, 8, 35.7, 42.1),
    (2048, 5120, 256, 16, 54.9, 62.4), (512, 7168, 256, 8, 59, 43),
])
def test_routers(T, d, E, k, direct, others):
    assert dispatch.route_direct(T, d, E, k) == (direct < others)


def test_routers_bounds():
    assert dispatch.route_direct(1, 256, 1, 1) and not dispatch.route_direct(0, 256, 1, 1)
    assert dispatch.route_direct(2048, 256, 32, 8) and not dispatch.route_direct(2049, 256, 32, 8)
    assert not dispatch.route_direct(64, 256, 100, 8)               # its columns do not align
    for E, k, T, last in ((72, 7, 64, 4608), (128, 8, 2048, 5120), (136, 3, 64, 3584), (256, 4, 1280, 4608),
                          (256, 4, 1281, 4096), (160, 15, 2048, 5120), (168, 15, 1951, 4608), (256, 16, 1281, 5120)):
        assert dispatch.route_direct(T, last, E, k) and not dispatch.route_direct(T, last + 256, E, k)


@pytest.mark.parametrize("K,E,rows,two,three", [
    # a forward with d = f = K, mean rows per expert
    (256, 64, 16, 24.8, 25.4), (256, 128, 16, 34.3, 35.3), (256, 128, 300, 76.5, 77.9), (256, 64, 900, 125.4, 127.2),
    (512, 64, 16, 44.7, 46.1), (512, 128, 100, 79.4, 81.1), (512, 128, 300, 163.9, 161.2), (512, 128, 900, 377.7, 368.2),
    (768, 64, 300, 182.4, 173.5), (768, 128, 900, 675.8, 660.9), (1024, 64, 16, 124.1, 118.7),
    (1024, 128, 300, 483.1, 474.1), (2048, 16, 100, 147.7, 136.7), (2048, 64, 900, 1699.6, 1664.8),
    # longer products, from 125 to 4096 rows (8 experts of 2048, d 7168, and 128 of 768, d 2048)
    (2048, 8, 125, 394, 369), (2048, 128, 512, 906, 878), (2048, 128, 1024, 1570, 1541), (2048, 8, 3000, 3580, 3607),
    (2048, 8, 4096, 4752, 4777),
])
def test_third_stage(K, E, rows, two, three):
    assert dispatch.deep_stages(K, rows * E, E) == (three < two)


def test_third_stage_bounds():
    assert dispatch.deep_stages(768, 1024 * 3, 3) and not dispatch.deep_stages(768, 1024 * 3 + 1, 3)
    assert dispatch.deep_stages(512, 600, 3) and not dispatch.deep_stages(512, 599, 3)
    assert not dispatch.deep_stages(256, 600, 3) and dispatch.deep_stages(768, 1, 0)


@pytest.mark.parametrize("d,f,E,rows,past,through", [
    (256, 512, 8, 6000, 150, 136), (256, 1024, 8, 1500, 87, 79), (256, 2048, 8, 1500, 139, 124), (512, 512, 32, 1500, 159, 157),
    (512, 1536, 8, 1500, 125, 113), (1024, 1024, 8, 1500, 116, 106), (1024, 2048, 8, 1500, 189, 186),
    (256, 512, 8, 1500, 56, 58), (512, 2048, 32, 256, 116, 122), (1024, 1536, 32, 256, 122, 134),
    (512, 1536, 32, 1500, 0.86, 1), (512, 1024, 8, 6000, 0.99, 1), (1024, 2048, 8, 6000, 0.93, 1),
    (2048, 1536, 8, 1500, 224, 232), (2048, 2048, 8, 1500, 263, 272),
])
def test_mx_kept_activations(d, f, E, rows, past, through):
    assert dispatch.mx_keep_l2(rows * E, E, d, f) == (through < past)
