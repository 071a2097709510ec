"""Convolutions of more results than the threads that a launch counts (32 bits along
an axis; of more, the launch runs what is left past a multiple of 2^32 and reports no
error).  Small whole numbers, so that every sum is exact in FP32 and BF16; planes at the
ends and in the middle of every channel are compared."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def memory_given_back():
    yield
    import torch
    torch.cuda.empty_cache()


def signs(shape, seed, dtype):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    out = torch.empty(shape, dtype=dtype, device="cuda")
    for n in range(shape[0]):
        for c in range(shape[1]):
            out[n, c] = torch.randint(-1, 2, shape[2:], generator=gen, device="cuda", dtype=torch.int8)
    return out


def weights(co, ci, K, dtype):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(5)
    return torch.randint(-3, 4, (co, ci, K, K, K), generator=gen, device="cuda").to(dtype)


def planes_equal(out, src, w, bias, flip):
    """out[n, r] = bias + sum of w over channels and taps of src, at four planes of each
    r; flip: w[channel, r] and the taps reversed (data gradient at stride 1)."""
    import torch
    K, n = w.shape[-1], src.shape[-1]
    p = K // 2
    for s in range(out.shape[0]):
        for r in range(out.shape[1]):
            for d in (0, 1, n // 2, n - 1):
                ref = torch.full((n, n), bias, device="cuda")
                for c in range(src.shape[1]):
                    slab = torch.zeros(K, n + 2 * p, n + 2 * p, device="cuda")
                    for k in range(K):
                        if 0 <= d + k - p < n:
                            slab[k, p:p + n, p:p + n] = src[s, c, d + k - p].float()
                    for k in np.ndindex(K, K, K):
                        tap = tuple(K - 1 - q for q in k) if flip else k
                        v = w[(c, r) + tap] if flip else w[(r, c) + tap]
                        ref += v.float() * slab[k[0], k[1]:k[1] + n, k[2]:k[2] + n]
                assert torch.equal(out[s, r, d].float(), ref), (s, r, d)


@pytest.mark.parametrize("N, Co", [(1, 2), (2, 1)])   # a thread per result; 16 rows a wave
def test_fp32_forward_past_a_launch(N, Co):
    import torch
    from paper_1504_08340_amd import binding as B
    n, K = 1291, 3                       # 2 n^3 = 2^32 + 8.3e6 results
    x, w = signs((N, 1, n, n, n), 3, torch.float32), weights(Co, 1, K, torch.float32)
    y = torch.full((N, Co, n, n, n), 7.0, device="cuda")
    b = torch.ones(Co, device="cuda")
    B.fwi_conv3d_forward(None, B.conv_shape(N, 1, n, n, n, Co, K, (1, 1, 1)), x, w, b, False, y)
    torch.cuda.synchronize()
    planes_equal(y, x, w, 1.0, False)


def test_fp32_data_gradient_past_a_launch():
    import torch
    from paper_1504_08340_amd import binding as B
    n, K = 1291, 3
    x, dy = signs((1, 2, n, n, n), 3, torch.float32), signs((1, 1, n, n, n), 4, torch.float32)
    w, dx = weights(1, 2, K, torch.float32), torch.full((1, 2, n, n, n), 7.0, device="cuda")
    dw, db = torch.empty_like(w), torch.empty(1, device="cuda")
    B.fwi_conv3d_backward(None, B.conv_shape(1, 2, n, n, n, 1, K, (1, 1, 1)), x, w, None, dy, False, dx, dw, db)
    torch.cuda.synchronize()
    planes_equal(dx, dy, w, 0.0, True)


@pytest.mark.parametrize("K, Ci, n", [(3, 1, 1025),    # the kernel for few channels, 4 n^3 = 2^32 + 1.3e7 threads
                                      (3, 5, 813)])    # the other, 8 n^3 = 2^32 + 4.0e6
def test_bf16_past_a_launch(K, Ci, n):
    import torch
    from paper_1504_08340_amd import binding as B
    x, w = signs((1, Ci, n, n, n), 3, torch.bfloat16), weights(1, Ci, K, torch.bfloat16)
    y = torch.full((1, 1, n, n, n), 7.0, device="cuda")
    b = torch.ones(1, device="cuda")
    B.fwi_conv3d_forward_bf16(None, B.conv_shape(1, Ci, n, n, n, 1, K, (1, 1, 1)), x, w, b, False, True, y)
    torch.cuda.synchronize()
    planes_equal(y, x, w, 1.0, False)


def test_bf16_more_positions_than_int():
    """2^31 + 4.2e6 positions of one sample."""
    import torch
    from paper_1504_08340_amd import binding as B
    n, K = 1291, 3
    x, w = signs((1, 1, n, n, n), 3, torch.bfloat16), weights(1, 1, K, torch.bfloat16)
    y = torch.full((1, 1, n, n, n), 7.0, device="cuda")
    B.fwi_conv3d_forward_bf16(None, B.conv_shape(1, 1, n, n, n, 1, K, (1, 1, 1)), x, w, None, False, True, y)
    torch.cuda.synchronize()
    planes_equal(y, x, w, 0.0, False)
