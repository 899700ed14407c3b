"""Which kernel a convolution runs: a function of the shape, asked on the host.  The lines are measured (beside the rules);
what is held here is on which side of them a shape falls."""
import pytest

F32, BF16 = 0, 1


def kernel(role, *shape):
    from paper_1901_06773_amd import binding as b
    return b.op_conv_kernel(role, *shape)


def test_unknown_and_refused_calls_have_no_kernel():
    assert kernel("fwd", 0, 8, 8, 3, 8, 3, 1, 1, F32) is None
    assert kernel("wgrad", 1, 8, 8, 3, 8, 3, 1, 1, 7) is None


# few input channels: too few groups of rows, or too few units in one, leave the per-element kernel ahead
@pytest.mark.parametrize("shape,fwd,wgrad", [
    ((2, 224, 224, 3, 64, 7, 2, 3, F32), False, False),
    ((6, 224, 224, 3, 64, 7, 2, 3, F32), False, False),
    ((8, 224, 224, 3, 64, 7, 2, 3, F32), False, True),       # 112 groups; 100 thousand positions
    ((16, 224, 224, 3, 64, 7, 2, 3, F32), True, True),
    ((32, 224, 224, 3, 64, 7, 2, 3, F32), True, True),
    ((32, 224, 224, 3, 64, 3, 1, 1, F32), True, False),      # 27 filter columns of 160
    ((2, 128, 128, 3, 128, 3, 1, 1, F32), False, False),
    ((256, 32, 32, 3, 64, 3, 1, 1, F32), False, False),      # four units for eight waves
    ((48, 224, 224, 3, 64, 4, 4, 0, F32), False, False),     # reads every value once
    ((2, 224, 224, 3, 64, 7, 2, 3, BF16), False, True),
    ((6, 224, 224, 3, 64, 7, 2, 3, BF16), True, True),
    ((1, 224, 224, 3, 64, 3, 1, 1, BF16), False, True),
    ((16, 32, 32, 3, 64, 3, 1, 1, BF16), False, True),
    ((1, 100, 100, 3, 64, 7, 2, 3, BF16), False, False),     # below 16384 positions
])
def test_few_channels(shape, fwd, wgrad):
    assert (kernel("fwd", *shape) == "smallc") == fwd
    assert (kernel("wgrad", *shape) == "smallc") == wgrad


# bf16 weight gradients: the tiling; 1x1 filters without a stride find a position's pixel without counting
@pytest.mark.parametrize("shape,name", [
    ((512, 14, 14, 256, 256, 3, 1, 1, BF16), "wgrad_bf16 256x128"),
    ((512, 7, 7, 512, 512, 3, 1, 1, BF16), "wgrad_bf16 256x128"),
    ((256, 28, 28, 512, 128, 1, 1, 0, BF16), "wgrad_bf16 128x256 plain"),
    ((64, 14, 14, 256, 256, 1, 1, 0, BF16), "wgrad_bf16 64x64 plain"),
    ((64, 14, 14, 256, 256, 1, 2, 0, BF16), "wgrad_bf16 64x64"),
    ((1, 4096, 4, 8, 8, 3, 1, 1, BF16), "wgrad_bf16 64x64"),
    ((1, 4097, 4, 8, 8, 3, 1, 1, BF16), "wgrad_bf16 64x64"),          # maps of any size
    ((8, 56, 56, 3, 64, 3, 1, 1, BF16), "smallc"),
    ((8, 56, 56, 12, 64, 3, 1, 1, BF16), "wgrad generic 64x64"),      # channels not in 8s
])
def test_bf16_weight_gradient(shape, name):
    assert kernel("wgrad", *shape) == name


def test_fp32_layers_reach_the_kernels_their_parity_tests_name():
    from test_gpu_x3 import CASES, WGRAD_CASES
    for n, h, w, cin, cout, r, stride, name in WGRAD_CASES:
        assert kernel("wgrad", n, h, w, cin, cout, r, stride, r // 2, F32) == name, (n, h, w, cin, cout)
    for n, h, w, cin, cout, r, stride, fwd, dgrad in CASES:
        shape = (n, h, w, cin, cout, r, stride, r // 2, F32)
        assert (kernel("fwd", *shape), kernel("dgrad", *shape)) == (fwd, dgrad), shape


# fp32: launches too small for the split products to pay, or bound by the result they write, stay with the fp32 instruction
@pytest.mark.parametrize("shape,name", [
    ((4, 56, 56, 256, 64, 1, 1, 0, F32), "igemm direct 64x64, two groups"),
    ((1, 128, 129, 256, 64, 1, 1, 0, F32), "igemm direct 64x64"),          # 258 tiles
    ((2, 8, 8, 224, 64, 1, 1, 0, F32), "igemm direct 64x64"),              # seven chunks of K: too short for two groups
    ((128, 56, 56, 64, 256, 1, 1, 0, F32), "igemm direct 64x64"),          # 411 MB of result, K of 64
    ((41, 14, 14, 256, 256, 3, 1, 1, F32), "igemm_x3_deep window 128x64"),
    ((32, 56, 56, 64, 256, 1, 1, 0, F32), "igemm direct 64x64"),           # writes four times what it reads
    ((41, 56, 56, 64, 256, 1, 1, 0, F32), "igemm direct 64x64"),
    ((41, 28, 28, 128, 512, 1, 1, 0, F32), "igemm_x3 128x128"),
    ((2, 9, 7, 288, 40, 1, 1, 0, F32), "igemm direct 64x64, two groups"),
    ((41, 14, 14, 100, 256, 3, 1, 1, F32), "igemm generic 64x64"),         # channels not in 16s, r > 1
])
def test_fp32_forward(shape, name):
    assert kernel("fwd", *shape) == name


def test_fp32_strided_data_gradients_reach_the_kernels_their_parity_tests_name():
    from test_gpu_strided_dgrad import CASES, KERNELS
    assert [kernel("dgrad", *c, F32) for c in CASES] == KERNELS


# fp32 weight gradients: small layers stay with the fp32 instruction where its kernel takes the shape
@pytest.mark.parametrize("shape,name", [
    ((1, 56, 56, 256, 64, 1, 1, 0, F32), "wgrad direct 64x64"),
    ((2, 7, 7, 512, 512, 3, 1, 1, F32), "wgrad direct 64x64"),
    ((41, 14, 14, 256, 256, 3, 1, 1, F32), "wgrad_x3 128x128"),
    ((41, 1, 1, 2048, 1000, 1, 1, 0, F32), "wgrad direct 64x64"),          # 41 positions
    ((1, 5000, 3, 64, 64, 3, 1, 1, F32), "wgrad fast 64x64"),              # rows beyond the float quotients
])
def test_fp32_weight_gradient(shape, name):
    assert kernel("wgrad", *shape) == name


# the numbers a launch profile reports: one keeps its kernel
@pytest.mark.parametrize("number,name", [
    (1, "igemm_kernel<generic>"), (2, "wgrad_kernel<fast>"), (3, "wgrad_kernel<generic>"), (4, "igemm_kernel<direct>"),
    (5, "wgrad_kernel<direct>"), (6, "wgrad_bf16_kernel"), (7, "igemm_bf16_kernel"), (8, "igemm_kernel<direct, two groups>"),
    (0, "?"), (15, "?"), (-1, "?"),
])
def test_numbers_of_the_kernels(number, name):
    import ctypes
    from paper_1901_06773_amd import binding as b
    f = b._lib._ZN3acc17conv_variant_nameEi
    f.restype, f.argtypes = ctypes.c_char_p, [ctypes.c_int]
    assert f(number).decode() == name


# bf16, strided filters: what is read is counted, not what the input holds
@pytest.mark.parametrize("shape,name", [
    ((125, 42, 39, 128, 256, 1, 2, 0, BF16), "igemm_bf16 256x256"),
    ((86, 26, 26, 512, 176, 1, 2, 0, BF16), "igemm_bf16 64x64"),
    ((41, 56, 56, 256, 512, 1, 2, 0, BF16), "igemm_bf16 256x256"),
    ((128, 56, 56, 128, 128, 3, 2, 1, BF16), "igemm_bf16 128x128"),
    ((32, 28, 28, 128, 128, 3, 2, 1, BF16), "igemm_bf16 64x64, four stages"),
])
def test_bf16_strided_filters(shape, name):
    assert kernel("fwd", *shape) == name
