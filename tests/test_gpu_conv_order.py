"""Order of k in the packed convolutions: channel groups and steps from tap to tap.

x3 on 256 x 256 tiles: channel groups of 64, 32, 16 and none, taps inside.  The other packed
shapes: channel counts below, at and above a panel's depth, which decide how a lane gets from
one panel's tap and channel to the next's.

Bit-exact on small integers against the FP64 convolution oracle (bars as in
test_gpu_conv.py), for channel counts of each group size with one and several groups,
filters of one tap and more, images smaller than the filter, and columns around one tile.
"""
import numpy as np
import pytest
import torch

from oracle import conv as OC

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("cin", [8, 16, 24, 32, 48, 64, 96, 192])
@pytest.mark.parametrize("R,image,cout", [(1, (2, 9, 15), 5), (3, (3, 11, 13), 257), (5, (5, 2, 3), 256),
                                          (7, (1, 20, 17), 30)])
def test_channel_groups(cin, R, image, cout):
    from paper_1804_10694_amd import tgemm as tg
    print(f"conv order cin={cin} R={R} {image} cout={cout}", flush=True)
    g = torch.Generator().manual_seed(cin + R)
    X = torch.randint(-4, 5, (*image, cin), generator=g).float()
    Wt = torch.randint(-4, 5, (R, R, cin, cout), generator=g).float()
    Y0 = torch.randint(-4, 5, (*image, cout), generator=g).float()
    ref = OC.conv2d(X, Wt, Y0, 1.5, 0.5)
    for runtime_r in (False, True):
        Y = Y0.to(DEV)
        tg.conv2d(X.to(DEV), Wt.to(DEV), Y, 1.5, 0.5, "x3", path="packed", shape=1, runtime_r=runtime_r)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(Y.cpu().numpy().astype(np.float64), ref.reshape(Y.shape))


@pytest.mark.parametrize("dtype,cin", [("f32", 4), ("f32", 8), ("f32", 12), ("f32", 16), ("f32", 20), ("f32", 32),
                                       ("f32", 36), ("x3", 8), ("x3", 16), ("x3", 24), ("x3", 32), ("x3", 40)])
@pytest.mark.parametrize("R", [1, 3, 5])
def test_panel_steps(dtype, cin, R):
    from paper_1804_10694_amd import tgemm as tg
    image, cout = (2, 13, 11), 20
    g = torch.Generator().manual_seed(100 * cin + R)
    X = torch.randint(-4, 5, (*image, cin), generator=g).float()
    Wt = torch.randint(-4, 5, (R, R, cin, cout), generator=g).float()
    Y0 = torch.randint(-4, 5, (*image, cout), generator=g).float()
    ref = OC.conv2d(X, Wt, Y0, 1.5, 0.5)
    for shape in range(4):
        print(f"conv steps {dtype} cin={cin} R={R} shape={shape}", flush=True)
        Y = Y0.to(DEV)
        tg.conv2d(X.to(DEV), Wt.to(DEV), Y, 1.5, 0.5, dtype, path="packed", shape=shape)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(Y.cpu().numpy().astype(np.float64), ref.reshape(Y.shape))


@pytest.mark.parametrize("image,cout", [((4, 45, 45), 256), ((4, 44, 45), 256), ((4, 45, 45), 255), ((1, 3, 5), 4)])
def test_auto_around_128_tiles(image, cout):
    from paper_1804_10694_amd import tgemm as tg
    g = torch.Generator().manual_seed(sum(image) + cout)
    X = torch.randint(-4, 5, (*image, 8), generator=g).float()
    Wt = torch.randint(-4, 5, (3, 3, 8, cout), generator=g).float()
    Y0 = torch.randint(-4, 5, (*image, cout), generator=g).float()
    print(f"conv auto {image} cout={cout}", flush=True)
    Y = Y0.to(DEV)
    tg.conv3x3(X.to(DEV), Wt.to(DEV), Y, 1.5, 0.5, "f32")
    torch.cuda.synchronize()
    np.testing.assert_array_equal(Y.cpu().numpy().astype(np.float64), OC.conv2d(X, Wt, Y0, 1.5, 0.5).reshape(Y.shape))
