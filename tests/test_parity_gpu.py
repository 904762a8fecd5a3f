"""Parity of the HIP path (through the C ABI) against the float64 oracle on the same seeded inputs.

Tolerance (fp32 path vs fp64 oracle): relative L2 error <= 1e-5 and max abs error <= 1e-4 * max|y|.
"""
import sys

import numpy as np
import pytest

from paper_2504_11681_amd import inputs

pytestmark = pytest.mark.gpu

REL_L2, MAX_ABS = 1e-5, 1e-4


@pytest.fixture(scope="module")
def gpu():
    import torch
    from paper_2504_11681_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.lib()   # fails loudly when the HIP library is missing
    return torch, binding


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def check(got: np.ndarray, want: np.ndarray, what="", rel_l2=REL_L2):
    got = got.astype(np.complex128)
    err = got - want
    rel = np.linalg.norm(err.ravel()) / np.linalg.norm(want.ravel())
    mx = np.max(np.abs(err)) / np.max(np.abs(want))
    say(f"   {what}: rel_l2={rel:.3e} max_abs/max|y|={mx:.3e}")
    assert rel <= rel_l2, f"{what}: relative L2 {rel:.3e}"
    assert mx <= MAX_ABS, f"{what}: max abs {mx:.3e}"


def close(got, want, what):
    """Both halves of the tolerance, silently (for the sweeps)."""
    err = np.asarray(got) - want
    rel = np.linalg.norm(err.ravel()) / np.linalg.norm(want.ravel())
    mx = np.max(np.abs(err)) / np.max(np.abs(want))
    assert rel <= REL_L2, f"{what}: relative L2 {rel:.3e}"
    assert mx <= MAX_ABS, f"{what}: max abs {mx:.3e}"


def writes_workspace(gpu, nbytes, call):
    """Whether call() writes to a registered workspace of nbytes: the kernels that keep their spectra there do, layers whose
    intermediates are held in y do not."""
    torch, binding = gpu
    ws = torch.full((nbytes,), 0x5A, dtype=torch.uint8, device="cuda")
    binding.set_workspace(ws)
    call()
    torch.cuda.synchronize()
    return bool((ws != 0x5A).any())


def run_gpu(gpu, fn_name, x, W, K):
    torch, binding = gpu
    xd = torch.from_numpy(x).cuda()
    Wd = torch.from_numpy(W).cuda()
    yd = torch.full((x.shape[0], W.shape[1]) + x.shape[2:], float("nan"), dtype=torch.complex64, device="cuda")
    getattr(binding, fn_name)(xd, Wd, yd, K)
    torch.cuda.synchronize()
    return yd.cpu().numpy()


def oracle_fn(oracle_mod, dims):
    return oracle_mod.spectral_conv1d if dims == 1 else oracle_mod.spectral_conv2d


# (B, C_in, C_out, N, K): several tiles, ragged channel counts, every supported N of the fused kernel
SMALL_1D = [
    (4, 16, 16, 64, 16),        # benchmark configuration 1
    (3, 5, 7, 64, 8),
    (2, 33, 40, 64, 64),        # K = N: no truncation
    (3, 9, 70, 128, 32),
    (2, 37, 17, 128, 128),
    (64, 64, 64, 256, 64),      # benchmark configuration 2
    (5, 19, 130, 256, 32),
    (2, 40, 33, 256, 16),
    (3, 24, 96, 256, 128),
    (3, 32, 96, 256, 64),       # whole channel blocks, but the last 128-output slab is only partly there
    (2, 64, 96, 128, 32),
    (2, 16, 160, 256, 32),
    (2, 20, 40, 256, 256),
    (3, 21, 66, 512, 64),
    (2, 35, 10, 512, 256),
    (2, 16, 100, 512, 32),
    (3, 13, 129, 1024, 128),
    (2, 20, 30, 1024, 32),
    (2, 9, 64, 1024, 256),
    (1, 1, 1, 1024, 64),
    (2, 32, 128, 1024, 128),
    (1, 48, 256, 1024, 64),
    (2, 16, 128, 1024, 128),
    (128, 16, 128, 1024, 64),   # half a chip of workgroups: the symmetric-wave kernel by default (below: the four-wave one)
    (70, 9, 130, 1024, 128),    # ... with masks (70 rows x 2 slabs)
    (130, 16, 64, 1024, 64),    # at most 64 outputs: the four-wave kernel whatever the batch
    (130, 16, 65, 1024, 64),    # one output more: the symmetric-wave kernel, slab half empty
]


@pytest.mark.parametrize("shape", SMALL_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
@pytest.mark.parametrize("fn", ["spectral_conv1d", "spectral_conv1d_staged"])
def test_1d_small(gpu, oracle_mod, fn, shape):
    B, Ci, Co, N, K = shape
    say(f"[case] {fn} {shape}")
    x = inputs.make_x(100 + N + K, B, Ci, (N,))
    W = inputs.make_W(100 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    got = run_gpu(gpu, fn, x, W, K)
    check(got, want, fn)


# unfused variant with pruned transforms (three kernels): narrow path N <= 256, wide path N = 1024
PRUNED_1D = [(4, 16, 16, 64, 16), (3, 5, 7, 64, 64), (2, 33, 40, 64, 32), (3, 9, 70, 128, 32), (2, 37, 17, 128, 128),
             (2, 5, 3, 128, 16), (64, 64, 64, 256, 64), (5, 19, 130, 256, 32), (2, 40, 33, 256, 16), (3, 24, 96, 256, 128),
             (2, 20, 40, 256, 256), (3, 13, 129, 1024, 128), (1, 1, 1, 1024, 64), (2, 20, 30, 1024, 64),
             (7, 3, 2, 256, 16),
             # 64 < C_in <= 128: the contraction with all of W resident in LDS (ragged channels and outputs, an odd
             # number of mode tiles, several tile pairs per workgroup, whole blocks)
             (5, 70, 65, 256, 64), (3, 97, 130, 1024, 128), (600, 128, 128, 256, 128), (9, 128, 64, 256, 128), (2, 100, 20, 128, 64),
             # long pencils (N1 x 256 decomposition): odd pencil counts, K / N1 from 16 to 256, no truncation
             (2, 5, 7, 2048, 128), (3, 3, 5, 2048, 256), (1, 1, 1, 2048, 2048), (2, 8, 8, 2048, 1024),
             (2, 6, 9, 4096, 256), (1, 3, 2, 4096, 1024), (1, 2, 2, 4096, 4096), (2, 33, 70, 4096, 512),
             (1, 4, 4, 2048, 512), (1, 2, 3, 4096, 2048),
             # the contraction's direct kernel (up to 512 workgroups or 32 outputs): channel counts around its steps and
             # blocks, either side of both limits, and each of the kernels past them
             (9, 8, 33, 256, 64), (9, 9, 31, 256, 64), (2, 17, 32, 128, 64), (3, 65, 40, 256, 128), (2, 129, 3, 256, 16),
             (260, 4, 32, 256, 256), (256, 33, 64, 256, 128), (257, 33, 64, 256, 128), (300, 20, 40, 256, 128), (260, 130, 40, 256, 128),
             (128, 129, 64, 256, 128), (129, 129, 64, 256, 128), (129, 128, 64, 256, 128),
             # fewer modes than the kernel's: cut spectra with several sweeps per workgroup, either side of the rule that
             # keeps all columns of a long pencil
             (600, 20, 40, 256, 100), (300, 17, 33, 1024, 100), (150, 9, 30, 2048, 150), (2, 5, 6, 2048, 448),
             (2, 5, 6, 2048, 449), (3, 3, 4, 4096, 900)]


@pytest.mark.parametrize("shape", PRUNED_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_pruned_variant(gpu, oracle_mod, shape):
    B, Ci, Co, N, K = shape
    say(f"[case] spectral_conv1d_pruned {shape}")
    x = inputs.make_x(300 + N + K, B, Ci, (N,))
    W = inputs.make_W(300 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d_pruned", x, W, K), want, "pruned")


# partially fused variants (FFT + CGEMM kernel then pruned inverse; pruned forward then CGEMM + iFFT kernel)
PARTIAL_1D = [(3, 20, 40, 256, 64), (2, 16, 128, 256, 32), (1, 33, 65, 256, 128), (2, 8, 32, 128, 32),
              (3, 13, 129, 128, 64), (2, 32, 64, 128, 128), (5, 1, 1, 256, 32), (2, 64, 96, 256, 128),
              (70, 16, 32, 256, 64)]


@pytest.mark.parametrize("fn", ["spectral_conv1d_fft_gemm", "spectral_conv1d_gemm_ifft"])
@pytest.mark.parametrize("shape", PARTIAL_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_partially_fused_variants(gpu, oracle_mod, shape, fn):
    B, Ci, Co, N, K = shape
    say(f"[case] {fn} {shape}")
    x = inputs.make_x(500 + N + K, B, Ci, (N,))
    W = inputs.make_W(500 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, fn, x, W, K), want, fn)


# per-shape dispatch: CGEMM + iFFT variant (C_out > 128 where it exists), fused kernel, pruned kernels for long
# pencils, staged path
AUTO_1D = [(2, 16, 256, 256, 64), (3, 20, 130, 128, 32), (2, 16, 64, 256, 64), (2, 9, 200, 1024, 128),
           (2, 4, 4, 2048, 100), (2, 5, 3, 256, 48), (2, 40, 300, 256, 128), (2, 9, 20, 4096, 512), (3, 5, 6, 2048, 256)]


@pytest.mark.parametrize("shape", AUTO_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_auto_dispatch(gpu, oracle_mod, shape):
    B, Ci, Co, N, K = shape
    say(f"[case] spectral_conv1d_auto {shape}")
    x = inputs.make_x(600 + N + K, B, Ci, (N,))
    W = inputs.make_W(600 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d_auto", x, W, K), want, "auto")


def random_shapes(seed, count):
    """Seeded random shapes (B, C_in, C_out, N, K) that every 1-D entry point accepts, small enough for the oracle."""
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(count):
        N = int(rng.choice([128, 256]))
        K = int(rng.choice([k for k in (32, 64, 128) if k <= N]))
        out.append((int(rng.integers(1, 6)), int(rng.integers(1, 80)), int(rng.integers(1, 300)), N, K))
    return out


@pytest.mark.parametrize("shape", random_shapes(2025, 12), ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_random_shapes_all_entry_points(gpu, oracle_mod, shape):
    """Every 1-D entry point on the same random shape (odd channel counts exercise all the masks)."""
    B, Ci, Co, N, K = shape
    x = inputs.make_x(700 + Ci + Co, B, Ci, (N,))
    W = inputs.make_W(700 + Ci + Co, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    for fn in ("spectral_conv1d", "spectral_conv1d_auto", "spectral_conv1d_pruned", "spectral_conv1d_fft_gemm",
               "spectral_conv1d_gemm_ifft", "spectral_conv1d_staged"):
        say(f"[case] {fn} random {shape}")
        check(run_gpu(gpu, fn, x, W, K), want, fn)


def test_1d_pruned_unsupported_shapes(gpu):
    torch, binding = gpu
    for (N, K) in [(512, 64), (32, 8), (1024, 200), (16, 16)]:
        x = torch.zeros((1, 2, N), dtype=torch.complex64, device="cuda")
        W = torch.zeros((2, 2), dtype=torch.complex64, device="cuda")
        y = torch.zeros((1, 2, N), dtype=torch.complex64, device="cuda")
        with pytest.raises(binding.TfnoError) as e:
            binding.spectral_conv1d_pruned(x, W, y, K)
        assert e.value.status == binding.ERR_UNSUPPORTED, (N, K)


STAGED_ONLY_1D = [(2, 3, 4, 2, 1), (2, 3, 4, 4, 3), (3, 6, 5, 32, 5), (2, 4, 4, 2048, 100), (1, 2, 3, 4096, 4096),
                  (2, 5, 3, 256, 48),
                  # lengths that are not powers of two (matrix transform; the shortest, which does not fit, direct sums)
                  (2, 3, 4, 3, 2), (3, 5, 4, 48, 12), (2, 4, 6, 421, 24), (1, 3, 2, 1000, 1000), (2, 2, 2, 85, 85),
                  (1, 2, 2, 4095, 7)]


@pytest.mark.parametrize("shape", STAGED_ONLY_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_staged_general_shapes(gpu, oracle_mod, shape):
    B, Ci, Co, N, K = shape
    say(f"[case] staged {shape}")
    x = inputs.make_x(7, B, Ci, (N,))
    W = inputs.make_W(7, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d_staged", x, W, K), want, "staged")


# grids of the image kernels (N in {64,128,256}, K in {16,32,64}), which few images go through as strips (the image kernels themselves: RECT_IMAGE
# and IMAGES_2D below), and other shapes of the strip pipeline
SMALL_2D = [(2, 3, 5, 64, 16), (1, 8, 8, 64, 8), (2, 5, 33, 128, 32), (1, 4, 3, 256, 64), (1, 2, 2, 64, 64),
            (1, 3, 2, 64, 32), (1, 3, 2, 128, 16), (2, 2, 2, 128, 64), (1, 2, 3, 256, 16), (1, 2, 2, 256, 32),
            (3, 7, 70, 256, 64), (1, 2, 2, 128, 128), (1, 2, 2, 512, 64)]


@pytest.mark.parametrize("shape", SMALL_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
@pytest.mark.parametrize("fn", ["spectral_conv2d", "spectral_conv2d_staged"])
def test_2d_small(gpu, oracle_mod, fn, shape):
    B, Ci, Co, N, K = shape
    say(f"[case] {fn} {shape}")
    x = inputs.make_x(200 + N + K, B, Ci, (N, N))
    W = inputs.make_W(200 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d(x, W, K)
    check(run_gpu(gpu, fn, x, W, K), want, fn)


def test_staged_lengths_that_are_not_powers_of_two(gpu, oracle_mod):
    """2-D staged twin on 85 x 48 and 421 x 12 grids, and the 1-D per-shape dispatch falling back to the staged path."""
    for (B, Ci, Co, N1, N2, K1, K2) in [(2, 3, 2, 85, 48, 12, 12), (1, 2, 3, 12, 421, 5, 20), (1, 2, 2, 64, 100, 16, 30)]:
        say(f"[case] staged rect {(B, Ci, Co, N1, N2, K1, K2)}")
        x = inputs.make_x(1500 + N1 + N2, B, Ci, (N1, N2))
        W = inputs.make_W(1500 + N1 + N2, Ci, Co)
        want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
        check(run_gpu_rect(gpu, "spectral_conv2d_rect_staged", x, W, K1, K2), want, "staged rect, any N")
    x = inputs.make_x(1501, 2, 3, (300,))
    W = inputs.make_W(1501, 3, 4)
    want, _ = oracle_mod.spectral_conv1d(x, W, 40)
    check(run_gpu(gpu, "spectral_conv1d_auto", x, W, 40), want, "auto, N = 300")


# the transforms that serve lengths with odd factors: remainders of their blocks of 16 pairs, edges of their tiles of 32 outputs, pencil
# counts around 32, sums dealt out to several waves, the direct sums of fields that do not fit (single kernels: MATDFT_FORMS,
# ROW_1D below).
# (B, C_in, C_out, N, K)
ODD_1D = [(1, 1, 1, 17, 17), (1, 2, 3, 127, 3), (2, 31, 33, 129, 31), (3, 11, 32, 144, 32), (1, 33, 1, 145, 33), (2, 5, 7, 257, 97),
          (1, 40, 24, 271, 128), (2, 17, 9, 390, 129), (700, 16, 48, 136, 72), (1100, 32, 30, 40, 40), (1, 3, 2, 3000, 65),
          (90, 3, 128, 100, 99), (2, 4, 4, 123, 123), (3, 20, 7, 64 + 1, 40), (2, 3, 3, 63, 63), (4, 300, 5, 56, 8), (3, 5, 6, 39, 39), (3, 5, 6, 41, 20),
          # many outputs (those of the matrix transform that store whole pencils: MATDFT_FORMS), lengths around 64, 128, 256 and 512
          (700, 2, 97, 65, 9), (700, 2, 97, 63, 9), (513, 2, 73, 127, 20), (300, 2, 91, 129, 17), (257, 2, 65, 255, 30),
          (200, 2, 91, 257, 12), (131, 2, 97, 511, 33), (131, 2, 97, 510, 33), (100, 2, 91, 513, 8)]


@pytest.mark.parametrize("shape", ODD_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_lengths_with_odd_factors(gpu, oracle_mod, shape):
    B, Ci, Co, N, K = shape
    say(f"[case] odd length {shape}")
    x = inputs.make_x(1550 + N + K, B, Ci, (N,))
    W = inputs.make_W(1550 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d_auto", x, W, K), want, "auto, odd length")


@pytest.mark.parametrize("shape", [(1024, 2, 16, 3, 2), (1024, 1, 16, 9, 2), (1024, 4, 16, 9, 2), (512, 9, 16, 7, 2)],
                         ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_short_odd_lengths_and_few_channels(gpu, oracle_mod, shape):
    """Hardly anything rounds here but the last step of each transform and every step of 8 channels of the contraction, 0.8 units
    of 2^-24 each when rounded downwards, and the roots and weights, 0.5 units each: 0.98e-7 up to 8 channels, 1.08e-7 up to 16;
    the bound is an eighth above that.  Leaving out the smallest partial products of the contraction, all of one sign,
    adds 2^-24.5 to the value itself: 1.2e-7 to 1.4e-7."""
    B, Ci, Co, N, K = shape
    say(f"[case] short odd length {shape}")
    x = inputs.make_x(1580 + N, B, Ci, (N,))
    W = inputs.make_W(1580 + N, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d_auto", x, W, K), want, "short odd length",
          rel_l2=1.125 * 2.0 ** -24 * np.sqrt((2 + (Ci + 7) // 8) * 0.64 + 3 * 0.25))


# (B, C_in, C_out, N1, N2, K1, K2): odd sides on either axis or both, one side a power of two
ODD_2D = [(2, 3, 2, 33, 31, 17, 16), (1, 2, 3, 3, 300, 2, 33), (2, 2, 2, 300, 5, 40, 5), (5, 7, 4, 64, 96, 64, 7), (3, 4, 5, 130, 32, 9, 32),
          (9, 16, 16, 85, 85, 12, 12), (1, 1, 1, 9, 7, 9, 7)]


@pytest.mark.parametrize("shape", ODD_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_sides_with_odd_factors(gpu, oracle_mod, shape):
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] odd sides {shape}")
    x = inputs.make_x(1560 + N1 + K2, B, Ci, (N1, N2))
    W = inputs.make_W(1560 + N1 + K2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    check(run_gpu_rect(gpu, "spectral_conv2d_rect_staged", x, W, K1, K2), want, "odd sides")


# Both sides odd: a workgroup per field, or a kernel per axis, by the rule on rounds and chains (tests/test_dispatch_rules.py).  (B, C_in, C_out, N1, N2,
# K1, K2): the shortest sides, both parities, one and two sixteens of modes on either axis, all parts of a sum and sets of waves, the last columns' tile
# full, with one column, with two; sides of equal length (one root table); long sums on either axis; and one step outside the kernel's sizes
FIELD_2D = [(32, 8, 8, 30, 30, 1, 1), (32, 8, 8, 31, 33, 15, 16), (32, 8, 9, 33, 34, 16, 17), (16, 17, 16, 33, 65, 17, 16), (32, 8, 8, 50, 66, 32, 32),
            (2, 3, 5, 85, 85, 12, 12), (8, 9, 40, 85, 85, 12, 12), (1, 2, 3, 60, 50, 9, 9), (1, 3, 2, 45, 97, 10, 11), (33, 32, 32, 40, 96, 8, 9),
            (8, 32, 33, 97, 129, 16, 20), (8, 32, 33, 63, 160, 17, 9), (4, 64, 65, 62, 255, 30, 31), (4, 128, 129, 62, 224, 30, 31), (4, 128, 128, 62, 225, 30, 31), (8, 32, 64, 220, 56, 25, 8), (8, 32, 63, 220, 56, 25, 8), (4, 64, 64, 36, 249, 9, 12), (16, 16, 16, 511, 41, 13, 9),
            (2, 128, 128, 500, 33, 32, 8), (2, 130, 128, 300, 130, 20, 21), (4, 33, 2, 194, 67, 16, 13),
            (32, 8, 8, 29, 33, 9, 9), (32, 8, 8, 33, 29, 9, 9), (32, 8, 8, 45, 45, 33, 9), (32, 8, 8, 45, 45, 9, 33), (16, 16, 16, 33, 257, 9, 9), (16, 16, 16, 513, 33, 9, 9),
            # (one side a power of two)
            (8, 2, 61, 128, 85, 12, 12), (8, 2, 61, 64, 200, 9, 10), (8, 2, 61, 64, 130, 9, 10)]


@pytest.mark.parametrize("shape", FIELD_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_fields_with_odd_sides(gpu, shape):
    """Bound: four sums on the matrix pipe (two axes, two directions), each with the rounding of its operands' sums and differences and
    of its own additions in blocks of 32 slots, at most 3 units of 2^-24 between them, and the contraction with 2: sqrt(4 9 + 4) 2^-24 = 3.8e-7."""
    torch, binding = gpu
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] field {shape}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1610 + N1 + K2)
    x = torch.randn((B, Ci, N1, N2), dtype=torch.complex64, device="cuda", generator=g)
    W = torch.randn((Ci, Co), dtype=torch.complex64, device="cuda", generator=g) / Ci ** 0.5
    y = torch.full((B, Co, N1, N2), float("nan"), dtype=torch.complex64, device="cuda")
    binding.spectral_conv2d_rect_staged(x, W, y, K1, K2)
    want = exact_layer(torch, x, W, K1, K2)
    rel = float((y - want).norm() / want.norm())
    worst = float((y - want).abs().max() / want.abs().max())
    say(f"   rel {rel:.2e}, max {worst:.2e}")
    assert rel <= 3.8e-7 and worst <= 4e-6, shape


# 1-D, few pencils: the forward kernel with 1 to 4 sixteens of modes per wave and several groups of them, one to eight waves to a sum, long sums,
# a last tile of pencils with one; the kernel that contracts and transforms back: channels past a step of eight, modes past a tile, one to eight
# tiles of modes (and shares of the channels), last slabs with one output and none missing, outputs in one group of workgroups and in
# several, as many waves as tiles of outputs (512 slabs and more); and shapes outside the rules.  (B, C_in, C_out, N, K)
ROW_1D = [(2, 3, 4, 33, 1), (3, 5, 33, 33, 33), (1, 17, 32, 34, 16), (3, 16, 31, 47, 17), (2, 9, 64, 63, 32), (5, 8, 65, 65, 33), (1, 1, 1, 66, 48), (3, 24, 40, 95, 49),
          (2, 40, 33, 97, 64), (2, 64, 32, 129, 65), (1, 65, 5, 255, 96), (2, 33, 40, 257, 97), (2, 64, 7, 300, 128), (1, 20, 12, 511, 160), (2, 3, 5, 600, 256), (2, 3, 5, 600, 257),
          (64, 40, 56, 1000, 50), (2, 15, 70, 1025, 12), (1, 128, 128, 1900, 20), (1, 4, 6, 4095, 7), (1, 4, 6, 3000, 200), (255, 64, 4, 90, 10), (256, 64, 4, 90, 10),
          (300, 9, 40, 33, 9), (512, 8, 32, 100, 20), (1024, 8, 24, 50, 9), (1024, 8, 23, 50, 9), (600, 4, 8, 50, 40), (530, 5, 30, 520, 9), (64, 64, 20, 200, 70), (65, 64, 20, 200, 70),
          (2, 129, 30, 130, 66), (129, 65, 32, 60, 33), (2, 4, 5, 31, 9)]


@pytest.mark.parametrize("shape", ROW_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_rows_with_odd_lengths(gpu, shape):
    """Bound: a sum on the matrix pipe each way, each with the rounding of its operands' sums and differences and of its own additions (those
    of the kernels beside these grow with the length: 3 units of 2^-24 and a sixteenth of one per block of 16 pairs), and the contraction with 3
    and one per 32 channels (single fields of few points, which run on direct sums: 2.8e-7 of 3.1e-7)."""
    torch, binding = gpu
    B, Ci, Co, N, K = shape
    say(f"[case] row {shape}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1620 + N + K)
    x = torch.randn((B, Ci, N), dtype=torch.complex64, device="cuda", generator=g)
    W = torch.randn((Ci, Co), dtype=torch.complex64, device="cuda", generator=g) / Ci ** 0.5
    y = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
    binding.spectral_conv1d_auto(x, W, y, K)
    want = exact_layer(torch, x[:, :, None], W, 1, K)[:, :, 0]
    rel = float((y - want).norm() / want.norm())
    worst = float((y - want).abs().max() / want.abs().max())
    bound = 2.0 ** -24 * np.sqrt(2 * (3 + N / 512) ** 2 + (3 + Ci / 32) ** 2)
    say(f"   rel {rel:.2e} of {bound:.2e}, max {worst:.2e}")
    assert rel <= bound and worst <= 10 * bound, shape


# Grids of powers of two with few images, whose strips are held in y: every pair of sides, one, two, four and eight input images to an output
# image's field (the last with rows to spare, and with none), ragged and whole slabs, the largest and smallest mode counts, and one step outside
# (no room for the input rows; more images than that: the image kernels).  (B, C_in, C_out, N1, N2, K1, K2)
FEW_IMAGES = [(2, 3, 5, 64, 64, 32, 32), (2, 5, 3, 64, 64, 16, 64), (1, 9, 4, 64, 128, 8, 9), (3, 7, 1, 64, 256, 4, 20), (1, 8, 1, 64, 64, 4, 16), (2, 9, 1, 64, 64, 4, 16),
              (2, 4, 3, 64, 64, 17, 12), (2, 33, 17, 128, 64, 32, 31), (2, 16, 4, 128, 128, 16, 64), (1, 17, 33, 128, 256, 64, 33), (2, 7, 2, 128, 64, 1, 1),
              (1, 16, 16, 256, 256, 64, 64), (2, 31, 4, 256, 64, 16, 16), (1, 5, 40, 256, 128, 33, 64), (1, 3, 2, 256, 256, 65, 40), (1, 2, 2, 256, 64, 128, 9), (1, 2, 2, 64, 64, 33, 9),
              (25, 22, 23, 64, 64, 9, 9), (26, 22, 23, 64, 64, 9, 9), (11, 17, 18, 256, 256, 9, 17), (12, 17, 18, 256, 256, 9, 17), (20, 14, 15, 128, 128, 30, 20), (10, 16, 13, 64, 256, 9, 60),
              (17, 35, 35, 64, 64, 16, 32), (10, 30, 30, 128, 128, 64, 64), (6, 40, 40, 256, 128, 32, 16), (40, 20, 20, 256, 64, 64, 32)]


@pytest.mark.parametrize("shape", FEW_IMAGES, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_few_and_many_images(gpu, shape):
    """Bound: up to 8 steps of butterflies along an axis, two axes, two directions, of about 0.7 units of 2^-24 each, and the contraction with
    3: sqrt(32 0.5 + 9) 2^-24 = 3.0e-7.  y begins 8 bytes past a line, between guards."""
    torch, binding = gpu
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] images {shape}")
    g = torch.Generator(device="cuda")
    g.manual_seed(1630 + N1 + K2)
    x = torch.randn((B, Ci, N1, N2), dtype=torch.complex64, device="cuda", generator=g)
    W = torch.randn((Ci, Co), dtype=torch.complex64, device="cuda", generator=g) / Ci ** 0.5
    n = B * Co * N1 * N2
    whole = torch.full((n + 2,), float("nan"), dtype=torch.complex64, device="cuda")
    y = whole[1:1 + n].view(B, Co, N1, N2)
    want = exact_layer(torch, x, W, K1, K2)
    for turn in range(2):                                   # (y holds the first call's result in the second)
        binding.spectral_conv2d_rect(x, W, y, K1, K2)
        rel = float((y - want).norm() / want.norm())
        worst = float((y - want).abs().max() / want.abs().max())
        say(f"   rel {rel:.2e}, max {worst:.2e}")
        assert rel <= 3.0e-7 and worst <= 3e-6, shape
    assert bool(torch.isnan(whole[:1].real).all()) and bool(torch.isnan(whole[n + 1:].real).all())


# (B, C_in, C_out, N1, N2, K1, K2), strips: layers that strips made slower (many retained rows) and layers that they serve
STRIPS_OR_IMAGES = [((45, 2, 10, 64, 128, 21, 3), False), ((59, 9, 15, 256, 64, 59, 2), False), ((25, 4, 26, 256, 128, 46, 19), False), ((14, 8, 18, 256, 256, 52, 3), False),
                    ((58, 2, 2, 64, 256, 19, 24), False), ((38, 2, 12, 64, 128, 23, 62), False), ((61, 2, 15, 128, 64, 27, 8), False),
                    ((19, 3, 18, 64, 128, 16, 6), True), ((26, 47, 13, 256, 64, 22, 23), True), ((1, 16, 16, 256, 256, 64, 64), True), ((8, 64, 64, 64, 64, 16, 16), True),
                    ((4, 64, 64, 64, 64, 33, 16), False), ((4, 32, 32, 256, 256, 64, 64), True)]


@pytest.mark.parametrize("shape,strips", STRIPS_OR_IMAGES, ids=str)
def test_2d_layers_of_few_images_by_strips_or_image_kernels(gpu, shape, strips):
    torch, binding = gpu
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] strips or images {shape}")
    x = torch.zeros((B, Ci, N1, N2), dtype=torch.complex64, device="cuda")
    W = torch.zeros((Ci, Co), dtype=torch.complex64, device="cuda")
    y = torch.empty((B, Co, N1, N2), dtype=torch.complex64, device="cuda")
    assert writes_workspace(gpu, binding.workspace_bytes_2d(0, *shape), lambda: binding.spectral_conv2d_rect(x, W, y, K1, K2)) == (not strips)


# Fused layers whose waves invert the slab they have accumulated without the workgroup's LDS (every wave a slab of 32 outputs and all modes): N 128
# and 256, four and eight waves, complex and real rows, whole and ragged slabs, a last one with one output, modes cut inside a built size.
# (entry, B, C_in, C_out, N, K)
OWN_SLABS = [("spectral_conv1d", 3, 32, 128, 128, 32), ("spectral_conv1d", 2, 33, 97, 128, 20), ("spectral_conv1d", 2, 64, 128, 128, 64), ("spectral_conv1d", 2, 20, 129, 128, 40),
             ("spectral_conv1d", 2, 32, 128, 128, 128), ("spectral_conv1d", 300, 33, 65, 128, 64), ("spectral_conv1d", 300, 32, 128, 128, 100), ("spectral_conv1d", 2, 32, 128, 256, 128),
             ("spectral_conv1d", 300, 17, 100, 256, 128), ("spectral_conv1d", 300, 16, 128, 256, 90), ("spectral_conv1d", 192, 32, 256, 256, 128), ("spectral_conv1d", 193, 40, 250, 256, 100),
             ("spectral_conv1d", 200, 9, 129, 256, 128), ("spectral_conv1d_real", 3, 32, 128, 128, 32), ("spectral_conv1d_real", 150, 21, 97, 128, 64),
             ("spectral_conv1d_real", 150, 32, 128, 256, 128), ("spectral_conv1d_real", 150, 9, 66, 256, 70)]


@pytest.mark.parametrize("case", OWN_SLABS, ids=lambda c: "%s_B%d_Ci%d_Co%d_N%d_K%d" % c)
def test_waves_that_own_their_slab(gpu, oracle_mod, case):
    torch, binding = gpu
    entry, B, Ci, Co, N, K = case
    say(f"[case] own slab {case}")
    x = inputs.make_x(1640 + N + K, B, Ci, (N,))
    W = inputs.make_W(1640 + N + K, Ci, Co)
    if entry == "spectral_conv1d":
        check(run_gpu(gpu, entry, x, W, K), oracle_mod.spectral_conv1d(x, W, K)[0], "own slab")
        return
    xr = np.ascontiguousarray(x.real)
    yd = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
    binding.spectral_conv1d_real(torch.from_numpy(xr).cuda(), torch.from_numpy(W).cuda(), yd, K)
    close(yd.cpu().numpy().astype(np.float64), oracle_mod.spectral_conv1d_real(xr, W, K)[0], case)


# 1024 points and few rows, spectra held in y: one, two and four input pencils to an output pencil, the last of them full and not, mode counts around
# the tiles of 32 and both built sizes, channels around the steps of 8 and 32, a last slab with one output; the limits of the rule (rows, modes, no
# room) on both sides.  (real, B, C_in, C_out, K)
ROWS_IN_Y = [(False, 1, 1, 1, 1), (False, 2, 33, 33, 64), (False, 3, 9, 5, 65), (False, 2, 20, 5, 17), (False, 2, 21, 5, 17), (False, 3, 40, 20, 128), (False, 2, 17, 64, 32),
             (False, 3, 130, 129, 100), (False, 97, 64, 64, 33), (False, 98, 64, 64, 33), (False, 2, 16, 16, 129), (True, 1, 1, 1, 1), (True, 2, 33, 33, 64), (True, 3, 9, 5, 65),
             (True, 3, 10, 5, 128), (True, 3, 11, 5, 128), (True, 2, 40, 70, 97), (True, 146, 64, 64, 128), (True, 147, 64, 64, 128)]


@pytest.mark.parametrize("case", ROWS_IN_Y, ids=lambda c: "%s_B%d_Ci%d_Co%d_K%d" % (("real" if c[0] else "complex",) + c[1:]))
def test_few_rows_of_1024_points(gpu, oracle_mod, case):
    """Bound: 10 steps of butterflies each way of about 0.7 units of 2^-24, and the contraction with 3 and one per 32 channels (130: 7 units):
    sqrt(20 0.5 + 49) 2^-24 = 4.5e-7."""
    torch, binding = gpu
    real, B, Ci, Co, K = case
    say(f"[case] rows in y {case}")
    x = inputs.make_x(1650 + Ci, B, Ci, (1024,))
    W = inputs.make_W(1650 + Ci, Ci, Co)
    dtype, call, want = torch.complex64, binding.spectral_conv1d_auto, None
    if real:
        x, dtype, call = np.ascontiguousarray(x.real), torch.float32, binding.spectral_conv1d_real
    want = (oracle_mod.spectral_conv1d_real if real else oracle_mod.spectral_conv1d)(x, W, K)[0]
    n, pad = B * Co * 1024, 2 if real else 1                # y begins 8 bytes past a line
    whole = torch.full((n + 2 * pad,), float("nan"), dtype=dtype, device="cuda")
    y = whole[pad:pad + n].view(B, Co, 1024)
    xd, Wd = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda()
    for turn in range(2):                                   # (y holds the first call's result in the second)
        call(xd, Wd, y, K)
        got = y.cpu().numpy()
        check(got.astype(np.float64 if real else np.complex128), want, "rows in y", rel_l2=4.5e-7)
    guards = torch.view_as_real(whole)[..., 0] if not real else whole
    assert bool(torch.isnan(guards[:pad]).all()) and bool(torch.isnan(guards[n + pad:]).all())


# Every form of the matrix transform, by the sides it reads and writes.  (B, C_in, C_out, N1, N2, K1, K2); N1 = 1: 1-D.  A form's direction is
# the inverse where its name says inverse or whole pencils, else the forward one; the test asserts that it is this kernel that runs, and
# not those of few pencils or of whole fields, which the last entries name.
MATDFT_FORMS = {
    "1-D, two output tiles per wave": (328, 100, 2, 1, 140, 1, 40), "1-D, three": (328, 100, 2, 1, 141, 1, 70), "1-D, four": (328, 100, 2, 1, 140, 1, 100),
    "1-D, long, two": (330, 100, 2, 1, 1030, 1, 64), "1-D, long, three": (330, 100, 2, 1, 1031, 1, 96), "1-D, long, four": (330, 100, 2, 1, 1030, 1, 128),
    "1-D, few points, two": (330, 100, 2, 1, 39, 1, 39), "1-D, four waves": (330, 50, 1, 1, 300, 1, 20), "1-D, long, four waves": (330, 50, 1, 1, 1030, 1, 20),
    "1-D, inverse": (3000, 1, 1, 1, 100, 1, 30), "1-D, inverse, two tiles": (33100, 1, 1, 1, 65, 1, 9), "1-D, long, inverse": (300, 1, 1, 1, 1410, 1, 40),
    "1-D, long, inverse, two tiles": (2800, 1, 1, 1, 1500, 1, 40), "1-D, whole pencils by one wave": (33100, 1, 1, 1, 127, 1, 20),
    "1-D, whole pencils by two waves": (33100, 1, 1, 1, 255, 1, 30), "1-D, whole pencils by four waves": (16600, 1, 1, 1, 511, 1, 33),
    "rows, two": (8, 63, 2, 66, 140, 5, 40), "rows, three": (8, 63, 2, 66, 141, 5, 70), "rows, four": (8, 63, 2, 66, 140, 5, 100),
    "rows, four waves": (2, 40, 3, 64, 140, 5, 20), "rows, eight waves": (2, 3, 4, 90, 300, 5, 20), "rows, few points, two": (8, 63, 2, 66, 39, 5, 39),
    "rows, long": (8, 49, 3, 21, 1500, 9, 20), "rows, long, two": (33, 100, 2, 10, 1100, 3, 50), "rows, long, four waves": (4, 49, 3, 21, 1500, 9, 20), "rows, long, eight waves": (1, 4, 3, 21, 1500, 9, 20),
    "rows, inverse in pieces, two tiles": (8, 2, 64, 64, 100, 7, 30), "rows, long, inverse, two tiles": (8, 2, 49, 9, 1500, 4, 20), "rows, long, inverse": (1, 2, 3, 9, 1500, 4, 20),
    "rows, whole pencils by one wave": (8, 2, 61, 128, 85, 12, 12), "rows, whole pencils by two waves": (8, 2, 61, 64, 200, 9, 10), "rows, whole pencils by two waves, just past 128": (8, 2, 130, 64, 130, 9, 10),
    "rows, whole pencils by four waves": (4, 2, 120, 61, 300, 9, 10), "rows, whole pencils by four waves, just past 256": (4, 2, 125, 70, 257, 9, 10),
    "rows, inverse in pieces, 300 points": (4, 2, 61, 61, 300, 9, 10), "rows, inverse in pieces, 257 points": (4, 2, 61, 70, 257, 9, 10),
    "rows, whole pencils by four waves, odd counts": (5, 2, 33, 67, 499, 5, 33),
    "columns, two": (28, 100, 2, 141, 13, 40, 12), "columns, three": (28, 100, 2, 141, 13, 70, 12), "columns, four": (28, 100, 2, 140, 13, 100, 12),
    "columns, four waves": (4, 50, 3, 141, 64, 20, 10), "columns, eight waves": (2, 3, 3, 301, 13, 20, 12), "columns, long": (33, 90, 3, 1050, 13, 20, 11),
    "columns, long, two": (33, 90, 2, 1050, 13, 50, 12), "columns, long, four waves": (8, 60, 3, 1500, 13, 20, 11), "columns, long, eight waves": (1, 6, 3, 1500, 13, 20, 11),
    "columns, inverse with two tiles": (28, 2, 100, 100, 12, 30, 12), "columns, long, inverse, two tiles": (8, 2, 49, 1500, 9, 20, 9),
    # the kernels of few pencils and of whole fields at the shapes of such forms
    "few pencils, 100 points": (330, 2, 100, 1, 100, 1, 30), "few pencils, 1500 points": (28, 2, 100, 1, 1500, 1, 40), "few pencils, a sum over eight waves": (8, 40, 8, 1, 1500, 1, 40),
    "few pencils, 40": (1, 40, 8, 1, 1500, 1, 40), "fields, 90 x 140": (2, 40, 40, 90, 140, 5, 20), "fields, 65 x 100": (8, 2, 64, 65, 100, 7, 30), "fields, 85 x 85": (8, 2, 73, 85, 85, 12, 12),
    "fields, 61 x 200": (8, 2, 61, 61, 200, 9, 10), "fields, 90 x 130": (8, 2, 61, 90, 130, 9, 10), "fields, 141 x 50": (4, 50, 60, 141, 50, 20, 10)}


def by_kernels_of_few_pencils_or_fields(binding, shape, inverse):
    """The library's own rules (internal functions, so by their mangled names)."""
    import ctypes
    B, Ci, Co, N1, N2, K1, K2 = shape
    name, args = (("_ZN4tfno17matgrid_supportedEixiiii", (+1 if inverse else -1, ctypes.c_longlong(B * (Co if inverse else Ci)), N1, N2, K1, K2)) if N1 > 1 else
                  ("_ZN4tfno24matrow_inverse_supportedExiiii", (ctypes.c_longlong(B), Ci, Co, N2, K2)) if inverse else
                  ("_ZN4tfno24matrow_forward_supportedExiii", (ctypes.c_longlong(B), Ci, N2, K2)))
    if N1 > 1 and (N1 & (N1 - 1) == 0 or N2 & (N2 - 1) == 0):
        return False                                        # (fields: both sides odd)
    fn = getattr(binding.lib(), name)
    fn.restype = ctypes.c_bool
    return fn(*args)


def exact_layer(torch, x, W, K1, K2):
    """The definition in float64 on the GPU, shared weights, as plain matrix products: x [B, C_in, N1, N2]."""
    B, Ci, N1, N2 = x.shape
    f1 = torch.from_numpy(np.exp(-2j * np.pi * (np.outer(np.arange(N1), np.arange(K1)) % N1) / N1)).cuda()
    f2 = torch.from_numpy(np.exp(-2j * np.pi * (np.outer(np.arange(N2), np.arange(K2)) % N2) / N2)).cuda()
    X = x.to(torch.complex128).reshape(-1, N2) @ f2
    X = X.reshape(B * Ci, N1, K2).transpose(1, 2).reshape(-1, N1) @ f1                                  # [B Ci K2, K1]
    Y = X.reshape(B, Ci, K2 * K1).transpose(1, 2).reshape(-1, Ci) @ W.to(torch.complex128)               # [B K2 K1, Co]
    Y = Y.reshape(B, K2, K1, -1).permute(0, 3, 1, 2).reshape(-1, K1) @ f1.conj().T.contiguous()         # [B Co K2, N1]
    y = Y.reshape(-1, K2, N1).transpose(1, 2).reshape(-1, K2) @ f2.conj().T.contiguous()
    return y.reshape(B, -1, N1, N2) / (N1 * N2)


@pytest.mark.parametrize("form", MATDFT_FORMS)
def test_forms_of_the_matrix_transform(gpu, form):
    """Tolerance: four times what 32-bit sums over these lengths measure (2.6e-7 at 1000 points, growing with the length)."""
    torch, binding = gpu
    B, Ci, Co, N1, N2, K1, K2 = MATDFT_FORMS[form]
    say(f"[case] matrix transform: {form} {MATDFT_FORMS[form]}")
    if form.startswith(("few pencils", "fields")):
        assert by_kernels_of_few_pencils_or_fields(binding, MATDFT_FORMS[form], False) and by_kernels_of_few_pencils_or_fields(binding, MATDFT_FORMS[form], True)
    else:
        assert not by_kernels_of_few_pencils_or_fields(binding, MATDFT_FORMS[form], "inverse" in form or "whole pencils" in form)
    gen = torch.Generator(device="cuda").manual_seed(1800 + N1 + N2)
    x = torch.view_as_complex(torch.randn((B, Ci, N1, N2, 2), generator=gen, device="cuda"))
    W = torch.view_as_complex(torch.randn((Ci, Co, 2), generator=gen, device="cuda")) / Ci ** 0.5
    y = torch.full((B, Co, N1, N2), float("nan"), dtype=torch.complex64, device="cuda")
    if N1 == 1:
        binding.spectral_conv1d_auto(x.reshape(B, Ci, N2), W, y.view(B, Co, N2), K2)
    else:
        binding.spectral_conv2d_rect_staged(x, W, y, K1, K2)
    want = exact_layer(torch, x, W, K1, K2)
    rel = ((y - want).norm() / want.norm()).item()
    say(f"   rel_l2={rel:.3e}")
    assert rel <= 1e-6 * max(1.0, max(N1, N2) / 1000)
    assert (y - want).abs().max().item() <= 1e-5 * want.abs().max().item()
    del x, y, want
    torch.cuda.empty_cache()


# One side a power of two, the other with odd factors: every transform that a power of two can take on either axis (column
# kernels with column counts around their 16, mode counts at and past what they take; pruned row kernels of every length
# with whole and cut spectra; the radix-2 transform of the lengths that have neither).  (C_in, C_out, N1, N2, K1, K2)
MIXED_2D = [(2, 3, 4096, 3, 4096, 3), (2, 3, 3, 4096, 3, 4096), (3, 2, 1024, 48, 1024, 48), (3, 2, 48, 1024, 48, 1024),
            (2, 2, 2048, 7, 2048, 7), (2, 2, 7, 2048, 7, 2048), (2, 2, 5, 2048, 5, 17), (2, 2, 6, 4096, 3, 500),
            (2, 2, 512, 13, 512, 6), (3, 3, 512, 33, 128, 33), (3, 3, 512, 31, 1, 15), (3, 3, 512, 48, 129, 20), (2, 2, 13, 512, 9, 300),
            (4, 3, 256, 25, 128, 16), (4, 3, 256, 25, 17, 17), (4, 3, 256, 25, 129, 1), (4, 3, 25, 256, 20, 33), (4, 3, 25, 256, 25, 256),
            (5, 4, 128, 100, 33, 48), (5, 4, 128, 9, 16, 9), (5, 4, 100, 128, 30, 20), (5, 4, 9, 128, 9, 128),
            (5, 4, 64, 96, 64, 7), (5, 4, 64, 96, 8, 96), (5, 4, 96, 64, 7, 64), (5, 4, 96, 64, 50, 9), (5, 4, 60, 1024, 12, 100),
            (5, 4, 16, 31, 16, 31), (5, 4, 31, 16, 31, 16), (3, 2, 31, 512, 5, 20), (2, 2, 9, 512, 9, 512), (2, 3, 7, 512, 3, 65),
            (2, 3, 7, 1024, 7, 129), (2, 2, 6, 1024, 3, 500), (5, 4, 2, 130, 1, 40), (5, 4, 130, 2, 40, 2), (3, 3, 32, 50, 20, 33)]


@pytest.mark.parametrize("shape", MIXED_2D, ids=lambda s: "Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_one_side_a_power_of_two(gpu, oracle_mod, shape):
    """The side that is a power of two keeps the error of a butterfly network, which grows with the square root of its depth:
    at most 12 steps each way of about 0.7 rounding units (2^-24), sqrt(24) 0.7 2^-24 = 2.0e-7, beside 1.5e-7 for the
    short other side and 1e-7 for the contraction: 2.7e-7 together; the bound is half as much again.  (One 32-bit sum over
    such a side gives 5e-7 at 1024 points and 1.1e-6 at 4096.)"""
    Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] mixed sides {shape}")
    x = inputs.make_x(1570 + N1 + K2, 2, Ci, (N1, N2))
    W = inputs.make_W(1570 + N1 + K2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    check(run_gpu_rect(gpu, "spectral_conv2d_rect_staged", x, W, K1, K2), want, "mixed sides", rel_l2=4e-7)


# (B, C_in, C_out, N1, N2, K1, K2): rows on the matrix pipe with one, four and eight waves to a sum and more tiles per wave
@pytest.mark.parametrize("shape", [(2, 2, 8, 4096, 3, 9, 3), (2, 3, 8, 4096, 39, 8, 5), (2, 2, 8, 1024, 150, 8, 20), (1, 2, 8, 1024, 300, 6, 8),
                                   (2, 8, 4, 4096, 70, 6, 40)], ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_rounding_offsets_do_not_gather_in_bin_zero(gpu, oracle_mod, shape):
    """The error of the lowest bin of the first axis is like that of the other kept bins.  Each is a sum of rounding errors
    over B C_out K2 >= 48 values: two such estimates differ by less than half; an offset common to all rows of a
    field adds up over N1 rows while the data add up to sqrt(N1), and made it 3 to 5 times the others'."""
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] offsets {shape}")
    x = inputs.make_x(1590 + N2, B, Ci, (N1, N2))
    W = inputs.make_W(1590 + N2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    err = run_gpu_rect(gpu, "spectral_conv2d_rect_staged", x, W, K1, K2) - want
    bins = np.sqrt(np.mean(np.abs(np.fft.fft(err, axis=2)[:, :, :K1]) ** 2, axis=(0, 1, 3)))
    say(f"   bin 0 / others: {bins[0] / np.sqrt(np.mean(bins[1:] ** 2)):.2f}")
    assert bins[0] <= 1.5 * np.sqrt(np.mean(bins[1:] ** 2)), shape


def test_2d_staged_general_shape(gpu, oracle_mod):
    B, Ci, Co, N, K = 2, 3, 2, 32, 5
    x = inputs.make_x(9, B, Ci, (N, N))
    W = inputs.make_W(9, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d(x, W, K)
    check(run_gpu(gpu, "spectral_conv2d_staged", x, W, K), want, "staged2d")


def run_image_kernels(gpu, x, W, K1, K2):
    """spectral_conv2d_rect, asserted to run the image kernels: few images go by strips held in y, which leave the workspace alone."""
    torch, binding = gpu
    B, Ci, N1, N2 = x.shape
    got = []
    need = binding.workspace_bytes_2d(0, B, Ci, W.shape[1], N1, N2, K1, K2)
    assert writes_workspace(gpu, need, lambda: got.append(run_gpu_rect(gpu, "spectral_conv2d_rect", x, W, K1, K2))), "not the image kernels"
    return got[0]


def run_gpu_rect(gpu, fn_name, x, W, K1, K2):
    torch, binding = gpu
    xd = torch.from_numpy(x).cuda()
    Wd = torch.from_numpy(W).cuda()
    yd = torch.full((x.shape[0], W.shape[1]) + x.shape[2:], float("nan"), dtype=torch.complex64, device="cuda")
    getattr(binding, fn_name)(xd, Wd, yd, K1, K2)
    torch.cuda.synchronize()
    return yd.cpu().numpy()


# every (N1, N2, K1, K2) instantiation of the image kernels: with nine input channels to one output there is no room for the
# strips of the input in y.  The same grids with 3 -> 2 channels go by strips where they fit.
RECT_IMAGE = [(n1, n2, k1, k2) for n1 in (64, 128, 256) for n2 in (64, 128, 256) for k1 in (16, 32, 64)
              for k2 in (16, 32, 64)]


@pytest.mark.parametrize("shape", RECT_IMAGE, ids=lambda s: "N%dx%d_K%dx%d" % s)
def test_2d_rect_image_kernels(gpu, oracle_mod, shape):
    N1, N2, K1, K2 = shape
    for B, Ci, Co in ((2, 3, 2), (2, 9, 1)):
        say(f"[case] spectral_conv2d_rect {shape} {(B, Ci, Co)}")
        x = inputs.make_x(300 + N1 + 2 * N2 + K1 + 3 * K2, B, Ci, (N1, N2))
        W = inputs.make_W(300 + N1 + 2 * N2 + K1 + 3 * K2, Ci, Co)
        want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
        check(run_image_kernels(gpu, x, W, K1, K2) if Ci == 9 else run_gpu_rect(gpu, "spectral_conv2d_rect", x, W, K1, K2), want, "rect")


# (B, C_in, C_out, N1, N2, K1, K2): the image kernels with ragged channels on every contraction kernel, with many images, with mode counts
# between the built sizes, and with more retained rows than strips have room for
IMAGES_2D = [(2, 9, 1, 64, 64, 12, 12), (1, 9, 2, 128, 256, 20, 48), (2, 9, 1, 256, 128, 64, 33), (40, 4, 4, 64, 256, 1, 5), (2, 33, 5, 256, 64, 64, 16), (4, 7, 70, 64, 256, 16, 64),
             (2, 66, 130, 128, 256, 32, 16), (6, 7, 70, 256, 256, 64, 64), (1, 1, 1, 64, 64, 33, 1), (2, 40, 33, 64, 64, 32, 32), (1, 130, 70, 128, 64, 64, 50), (1, 257, 9, 64, 64, 40, 9)]


@pytest.mark.parametrize("shape", IMAGES_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_image_kernels(gpu, oracle_mod, shape):
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] image kernels {shape}")
    x = inputs.make_x(350 + N1 + K2, B, Ci, (N1, N2))
    W = inputs.make_W(350 + N1 + K2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    check(run_image_kernels(gpu, x, W, K1, K2), want, "image kernels")


# (B, C_in, C_out, N1, N2, K1, K2): ragged channels on grids of the image kernels, strip-pipeline shapes (first axis or mode
# count outside the image kernels' set), and shapes only the staged twin takes
RECT_MIXED = [(3, 7, 70, 64, 256, 16, 64), (2, 33, 5, 256, 64, 64, 16), (1, 66, 130, 128, 256, 32, 16),
              (2, 3, 4, 32, 256, 8, 64), (1, 2, 3, 512, 64, 100, 16), (2, 3, 2, 16, 1024, 16, 128),
              (1, 2, 2, 1024, 128, 64, 128), (2, 2, 3, 2, 64, 1, 8)]
RECT_STAGED_ONLY = [(2, 3, 2, 8, 32, 3, 5), (1, 2, 2, 64, 16, 64, 16), (2, 2, 3, 128, 4, 7, 2), (1, 1, 1, 2, 2048, 2, 100)]


@pytest.mark.parametrize("shape", RECT_MIXED, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
@pytest.mark.parametrize("fn", ["spectral_conv2d_rect", "spectral_conv2d_rect_staged"])
def test_2d_rect_mixed(gpu, oracle_mod, fn, shape):
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] {fn} {shape}")
    x = inputs.make_x(400 + N1 + K2, B, Ci, (N1, N2))
    W = inputs.make_W(400 + N1 + K2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    check(run_gpu_rect(gpu, fn, x, W, K1, K2), want, fn)


# the paper's 2-D pipeline on request: image-kernel shapes (where the default entry point takes the other path), shapes
# it serves anyway, modes between the built sizes on both axes
STRIPS_2D = [(3, 7, 70, 64, 256, 16, 64), (2, 33, 5, 256, 64, 64, 16), (2, 8, 8, 64, 64, 16, 16), (2, 3, 4, 32, 256, 8, 64),
             (1, 5, 3, 128, 128, 20, 12), (2, 16, 16, 256, 256, 64, 64)]


@pytest.mark.parametrize("shape", STRIPS_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_strip_pipeline_on_request(gpu, oracle_mod, shape):
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] spectral_conv2d_strips {shape}")
    x = inputs.make_x(450 + N1 + K2, B, Ci, (N1, N2))
    W = inputs.make_W(450 + N1 + K2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    check(run_gpu_rect(gpu, "spectral_conv2d_strips", x, W, K1, K2), want, "strips")


# column kernels along the first axis: every length, mode counts at and one past the multiples of their first radix (8 for
# 64 rows, else 16) where the pruned stage changes, the largest they take and one more (staged transform)
COLS_2D = [(n1, k1) for n1, p in ((64, 8), (128, 16), (256, 16), (512, 16)) for k1 in (1, p, p + 1, 2 * p + 1, 4 * p + 1, 8 * p, 8 * p + 1)
           if k1 <= n1]


@pytest.mark.parametrize("shape", COLS_2D, ids=lambda s: "N%d_K%d" % s)
def test_2d_strip_pipeline_column_kernels(gpu, oracle_mod, shape):
    N1, K1 = shape
    say(f"[case] column kernels {shape}")
    x = inputs.make_x(460 + N1 + K1, 2, 3, (N1, 64))
    W = inputs.make_W(460 + N1 + K1, 3, 2)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, 10)
    check(run_gpu_rect(gpu, "spectral_conv2d_strips", x, W, K1, 10), want, "column kernels")


@pytest.mark.parametrize("K1", [1, 2])
def test_2d_strip_pipeline_few_modes_of_long_columns(gpu, oracle_mod, K1):
    """The second stage of the column kernels sums 32 terms for one or two modes of 512 rows, 8 terms for 64 rows.  In one
    chain these round by 1.06e-7 and 0.56e-7, in blocks of four by 0.70e-7 and 0.49e-7 (rms of such sums of normal
    values); beside the rest of the layer, 1.5e-7, that is a ratio of 1.14 between the two column lengths, or 1.05."""
    errs = []
    for N1 in (64, 512):
        x = inputs.make_x(490 + N1, 8, 16, (N1, 64))
        W = inputs.make_W(490 + N1, 16, 16)
        want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, 16)
        got = run_gpu_rect(gpu, "spectral_conv2d_strips", x, W, K1, 16)
        errs.append(np.linalg.norm(got - want) / np.linalg.norm(want))
    say(f"   K1 = {K1}: 64 rows {errs[0]:.3e}, 512 rows {errs[1]:.3e}, ratio {errs[1] / errs[0]:.3f}")
    assert errs[1] <= 1.1 * errs[0]


@pytest.mark.parametrize("shape", RECT_STAGED_ONLY, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_rect_staged_general_shapes(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] staged rect {shape}")
    x = inputs.make_x(500 + N1 + K2, B, Ci, (N1, N2))
    W = inputs.make_W(500 + N1 + K2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    check(run_gpu_rect(gpu, "spectral_conv2d_rect_staged", x, W, K1, K2), want, "staged rect")
    with pytest.raises(binding.TfnoError) as e:
        run_gpu_rect(gpu, "spectral_conv2d_rect", x, W, K1, K2)
    assert e.value.status == binding.ERR_UNSUPPORTED


def test_2d_rect_square_case_is_bitwise_the_square_entry_point(gpu):
    for Ci, Co in ((5, 6), (9, 1)):                         # strips held in y, image kernels
        x = inputs.make_x(77, 2, Ci, (128, 128))
        W = inputs.make_W(77, Ci, Co)
        a = run_image_kernels(gpu, x, W, 32, 32) if Ci == 9 else run_gpu_rect(gpu, "spectral_conv2d_rect", x, W, 32, 32)
        b = run_gpu(gpu, "spectral_conv2d", x, W, 32)
        assert np.array_equal(a.view(np.float32), b.view(np.float32))


# per-mode weights (B, C_in, C_out, N, K): several batch groups, ragged channels, K below / equal / above one tile
PERMODE_1D = [(4, 16, 16, 64, 16), (19, 5, 7, 64, 64), (9, 33, 40, 128, 32), (3, 9, 70, 128, 128), (17, 6, 18, 256, 256),
              (1, 1, 1, 256, 16), (2, 20, 30, 1024, 64), (11, 13, 17, 1024, 128), (8, 3, 2, 256, 128),
              # mode counts between the built sizes (weights hold exactly K matrices)
              (3, 5, 7, 64, 12), (9, 9, 4, 256, 100), (4, 6, 6, 1024, 72), (2, 3, 3, 128, 1),
              # batches and output counts that fill 64 x 64 tiles per mode (ragged last tiles, channel mask, surplus modes)
              (250, 16, 128, 256, 128), (256, 9, 120, 256, 100),
              # the contraction's kernels on both sides of the rules: matrix pipe with and without masks at fewer than 128
              # modes and at counts that are no multiple of 8 (joint tiles shared by batch elements), FP32 with 8 x 8, 4 x 4,
              # 2 x 2 and 1 x 1 results per thread, C_in not a multiple of the channels in flight
              (96, 16, 64, 64, 64), (64, 24, 160, 128, 40), (71, 20, 50, 256, 117), (260, 9, 131, 256, 128), (33, 15, 65, 256, 33),
              (5, 33, 9, 1024, 17), (2, 7, 3, 64, 3)]


@pytest.mark.parametrize("shape", PERMODE_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_permode(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N, K = shape
    say(f"[case] spectral_conv1d_permode {shape}")
    x = inputs.make_x(700 + N + K, B, Ci, (N,))
    W = np.ascontiguousarray(inputs.make_W(700 + N + K, Ci, Co * K).reshape(Ci, Co, K))
    want, _ = oracle_mod.spectral_conv1d_permode(x, W)
    xd, Wd = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda()
    yd = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
    binding.spectral_conv1d_permode(xd, Wd, yd)
    torch.cuda.synchronize()
    check(yd.cpu().numpy(), want, "permode 1d")


# (B, C_in, C_out, N1, N2, K1, K2)
PERMODE_2D = [(2, 3, 5, 64, 64, 16, 16), (9, 5, 33, 128, 64, 32, 16), (1, 4, 3, 256, 256, 64, 64), (10, 2, 2, 64, 256, 16, 64),
              (3, 17, 9, 128, 128, 64, 32), (2, 3, 4, 64, 128, 12, 20), (9, 2, 3, 256, 64, 33, 5),
              (120, 20, 112, 64, 64, 16, 16), (40, 16, 33, 64, 64, 15, 21), (32, 32, 32, 64, 64, 24, 16)]


@pytest.mark.parametrize("shape", PERMODE_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_permode(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] spectral_conv2d_permode {shape}")
    x = inputs.make_x(800 + N1 + K2, B, Ci, (N1, N2))
    W = np.ascontiguousarray(inputs.make_W(800 + N1 + K2, Ci, Co * K1 * K2).reshape(Ci, Co, K1, K2))
    want, _ = oracle_mod.spectral_conv2d_permode(x, W)
    xd, Wd = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda()
    yd = torch.full((B, Co, N1, N2), float("nan"), dtype=torch.complex64, device="cuda")
    binding.spectral_conv2d_permode(xd, Wd, yd)
    torch.cuda.synchronize()
    check(yd.cpu().numpy(), want, "permode 2d")


@pytest.mark.parametrize("shape", [(16, 512, 64, 256, 128), (16, 300, 27, 256, 81), (3, 512, 5, 64, 16), (64, 512, 20, 64, 24)],
                         ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_permode_sums_over_many_channels(gpu, oracle_mod, shape):
    """Small per-mode products on the FP32 kernel: sums of at most 16 channels are added up, so that the rounding grows with
    sqrt(16) + sqrt(C / 16) terms' worth of 2^-24 / sqrt(6) each (about 2e-7 at 512 channels, beside 1.6e-7 for the two
    transforms; the bound is half as much again) and not with sqrt(2 C), which measured 6e-7."""
    B, Ci, Co, N, K = shape
    say(f"[case] many channels {shape}")
    x = inputs.make_x(1650 + Ci, B, Ci, (N,))
    W = np.ascontiguousarray(inputs.make_W(1650 + Ci, Ci, Co * K).reshape(Ci, Co, K))
    f = np.exp(-2j * np.pi * np.outer(np.arange(N), np.arange(K)) / N)
    X = x.astype(np.complex128) @ f
    want = np.matmul(X.transpose(2, 0, 1), W.astype(np.complex128).transpose(2, 0, 1)).transpose(1, 2, 0) @ np.conj(f.T) / N
    torch, binding = gpu
    yd = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
    binding.spectral_conv1d_permode(torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), yd)
    check(yd.cpu().numpy(), want, "per mode", rel_l2=3.8e-7)


# Layers whose truncated spectra pass through the workspace, with fewer modes than the kernels' (all bins stored, or only the
# kept ones rounded up to 8), by the FP32 and the matrix-pipe contraction: modes that are not kept, and the rest of the last
# 128-mode tile, hold whatever the workspace held unless a kernel writes them.  (entry, B, C_in, C_out, N, K)
SURPLUS = [(e, B, ci, co, n, k) for e in ("spectral_conv1d_permode", "fno1d_real")
           for B, ci, co, n, k in ((5, 7, 9, 256, 121), (5, 7, 9, 256, 100), (64, 32, 64, 256, 123), (64, 32, 64, 256, 99),
                                   (3, 5, 6, 64, 9), (3, 5, 6, 64, 5), (2, 9, 4, 1024, 62), (3, 4, 4, 128, 60))] + [
    (e, B, ci, co, n, k) for e in ("spectral_conv1d_pruned", "spectral_conv1d_fft_gemm", "spectral_conv1d_gemm_ifft")
    for B, ci, co, n, k in ((5, 7, 9, 256, 121), (5, 7, 9, 256, 51), (9, 40, 33, 128, 57), (9, 40, 33, 128, 20))] + [
    ("spectral_conv1d_pruned", 3, 4, 5, 2048, 150), ("spectral_conv1d_pruned", 3, 4, 5, 2048, 500), ("spectral_conv1d_pruned", 3, 4, 5, 1024, 127)]


@pytest.mark.parametrize("case", SURPLUS, ids=lambda c: "%s-B%d_Ci%d_Co%d_N%d_K%d" % c)
def test_what_the_workspace_held_does_not_matter(gpu, oracle_mod, case):
    torch, binding = gpu
    entry, B, Ci, Co, N, K = case
    say(f"[case] surplus modes {case}")
    real, per_mode = entry == "fno1d_real", entry in ("fno1d_real", "spectral_conv1d_permode")
    x = inputs.make_x(1600 + N + K, B, Ci, (N,))
    W = inputs.make_W(1600 + N + K, Ci, Co * K if per_mode else Co)
    if real:
        x = np.ascontiguousarray(x.real)
    if per_mode:
        W = W.reshape(Ci, Co, K)
    f = np.exp(-2j * np.pi * np.outer(np.arange(N), np.arange(K)) / N)
    X = x.astype(np.complex128) @ f
    Y = np.einsum("bck,cok->bok", X, W) if per_mode else np.einsum("bck,co->bok", X, W)
    if real:
        Y[:, :, 0] *= 0.5
    want = Y @ np.conj(f.T) / N
    want = 2 * want.real if real else want
    xd, Wd = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda()
    yd = torch.full((B, Co, N), float("nan"), dtype=xd.dtype, device="cuda")
    junk = torch.full((1 << 24,), 0xff, dtype=torch.uint8, device="cuda")       # NaN in every word
    binding.set_workspace(junk)
    try:
        getattr(binding, entry)(xd, Wd, yd) if per_mode else getattr(binding, entry)(xd, Wd, yd, K)
        torch.cuda.synchronize()
    finally:
        binding.set_workspace(None)
    check(yd.cpu().numpy(), want, entry)


def test_large_batch_uses_64_bit_offsets(gpu, oracle_mod):
    """B = 2^18 (1 GiB tensors, 2^18 workgroups): sampled batch elements against the oracle, including the last, whose
    byte offset is past 2^31; the rest of the batch is filled on the device and only checked to be written."""
    torch, binding = gpu
    B, Ci, Co, N, K = 1 << 18, 8, 8, 64, 16
    say(f"[case] large batch 1-D B={B}")
    gen = torch.Generator(device="cuda").manual_seed(5)
    xd = torch.view_as_complex(torch.randn((B, Ci, N, 2), generator=gen, device="cuda", dtype=torch.float32))
    Wn = inputs.make_W(5, Ci, Co)
    sample = [0, 1, B // 2 + 3, B - 1]
    for b in sample:
        xd[b] = torch.from_numpy(inputs.make_x_element(5, b, Ci, (N,))).cuda()
    Wd = torch.from_numpy(Wn).cuda()
    for fn in ("spectral_conv1d", "spectral_conv1d_pruned"):
        yd = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
        getattr(binding, fn)(xd, Wd, yd, K)
        torch.cuda.synchronize()
        assert not torch.isnan(torch.view_as_real(yd)).any().item(), "some outputs were never written"
        for b in sample:
            want, _ = oracle_mod.spectral_conv1d(inputs.make_x_element(5, b, Ci, (N,))[None], Wn, K)
            check(yd[b].cpu().numpy()[None], want, f"{fn} b={b}")
        del yd
    del xd
    torch.cuda.empty_cache()


def test_contraction_of_more_tiles_than_one_launch_takes(gpu):
    """2^24 tiles of 128 modes: a launch has fewer than 2^32 threads, so one workgroup of 256 threads per tile is not possible
    and the contraction has to take a kernel that walks several tiles.  All modes are kept and there is one channel, so
    y = W x; 32-bit rounding of two transforms of 64 points leaves a few 1e-7."""
    torch, binding = gpu
    B = 1 << 25
    say("[case] 2^24 contraction tiles, 69 GB")
    if torch.cuda.mem_get_info()[0] < (80 << 30):
        pytest.skip("needs 80 GB of free device memory")
    binding.set_workspace(None)
    block = torch.randn(1 << 16, 1, 64, dtype=torch.complex64, device="cuda")
    x = block.repeat(B >> 16, 1, 1)
    W = torch.full((1, 1), 0.75 - 0.5j, dtype=torch.complex64, device="cuda")
    y = torch.empty_like(x)
    try:
        binding.spectral_conv1d_pruned(x, W, y, 64)
        torch.cuda.synchronize()
        want = block.to(torch.complex128) * (0.75 - 0.5j)
        for first in (0, B // 2 - (1 << 15), B - (1 << 16)):
            part = y[first:first + (1 << 16)].to(torch.complex128)
            err = (part - want.roll(-(first & 0xffff), 0)).norm() / want.norm()
            say(f"   rows from {first}: {err.item():.2e}")
            assert err.item() <= 1e-6
    finally:
        binding.set_workspace(None)
        del x, y
        torch.cuda.empty_cache()


def test_many_small_images_2d(gpu, oracle_mod):
    """32768 images of 64 x 64 (1 GiB): sampled batch elements against the oracle."""
    torch, binding = gpu
    B, Ci, Co, N, K = 4096, 8, 8, 64, 16
    say(f"[case] many images 2-D B={B}")
    gen = torch.Generator(device="cuda").manual_seed(6)
    xd = torch.view_as_complex(torch.randn((B, Ci, N, N, 2), generator=gen, device="cuda", dtype=torch.float32))
    Wn = inputs.make_W(6, Ci, Co)
    sample = [0, B // 3, B - 1]
    for b in sample:
        xd[b] = torch.from_numpy(inputs.make_x_element(6, b, Ci, (N, N))).cuda()
    Wd = torch.from_numpy(Wn).cuda()
    yd = torch.full((B, Co, N, N), float("nan"), dtype=torch.complex64, device="cuda")
    binding.spectral_conv2d(xd, Wd, yd, K)
    torch.cuda.synchronize()
    assert not torch.isnan(torch.view_as_real(yd)).any().item(), "some outputs were never written"
    for b in sample:
        want, _ = oracle_mod.spectral_conv2d(inputs.make_x_element(6, b, Ci, (N, N))[None], Wn, K)
        check(yd[b].cpu().numpy()[None], want, f"2d b={b}")
    del xd, yd
    torch.cuda.empty_cache()


def test_entry_points_replay_from_a_hip_graph(gpu):
    """The entry points only enqueue kernels on the caller's stream, so they can be captured once their first (eager)
    call has been made: three replays, with eager work and synchronisation in between, each bitwise equal to eager.  The fused 1-D
    layer; the 2-D layer by image kernels and by strips held in y; rows of 1024 points, complex and real, whose spectra are held in y."""
    torch, binding = gpu
    say("[case] HIP graph capture of the fused 1-D, the 2-D and the few-rows entry points")
    layers = []
    for call, B, Ci, Co, dims, K in ((binding.spectral_conv1d, 8, 24, 40, (256,), (64,)), (binding.spectral_conv2d_rect, 2, 9, 1, (64, 128), (40, 32)),
                                     (binding.spectral_conv2d_rect, 2, 5, 6, (64, 128), (16, 32)), (binding.spectral_conv1d_auto, 4, 24, 40, (1024,), (50,)),
                                     (binding.spectral_conv1d_real, 4, 24, 40, (1024,), (50,))):
        x = inputs.make_x(11 + len(layers), B, Ci, dims)
        if call is binding.spectral_conv1d_real:
            x = np.ascontiguousarray(x.real)
        x = torch.from_numpy(x).cuda()
        layers.append((call, x, torch.from_numpy(inputs.make_W(11 + len(layers), Ci, Co)).cuda(), torch.zeros((B, Co) + dims, dtype=x.dtype, device="cuda"), K))

    def run(layer, *stream):
        call, x, W, y, K = layer
        call(x, W, y, *K, *stream)

    # (which of them use the workspace: the image kernels alone.  One buffer for all, registered before the capture)
    need = binding.workspace_bytes_2d(0, 2, 9, 1, 64, 128, 40, 32) + binding.workspace_bytes_2d(0, 2, 5, 6, 64, 128, 16, 32)
    assert [writes_workspace(gpu, need, lambda: run(layer)) for layer in layers] == [False, True, False, False, False]
    want = [y.clone() for _, _, _, y, _ in layers]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            for layer in layers:
                run(layer, torch.cuda.current_stream().cuda_stream)
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        for layer in layers:
            layer[3].zero_()
        run(layers[1])                                      # (eager work between the replays)
        layers[1][3].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for layer, w in zip(layers, want):
            assert torch.equal(layer[3], w)


def test_general_layers_replay_from_a_hip_graph(gpu):
    """The same for odd lengths, odd and mixed grids, the column kernels and the per-mode layers: captured after one eager
    call each, replayed three times with eager work between, results the same bits."""
    torch, binding = gpu
    say("[case] HIP graph capture of odd lengths, mixed grids, column kernels, per-mode layers")
    layers = []
    for name, B, Ci, Co, dims, K in (("spectral_conv1d_auto", 9, 24, 40, (1000,), (50,)), ("spectral_conv2d_rect_staged", 2, 5, 6, (85, 90), (12, 9)),
                                     ("spectral_conv2d_rect_staged", 2, 5, 6, (85, 64), (12, 9)), ("spectral_conv2d_rect_staged", 2, 5, 6, (30, 512), (12, 40)),
                                     ("spectral_conv2d_rect_staged", 2, 5, 6, (128, 25), (12, 9)), ("spectral_conv2d_rect_staged", 2, 5, 6, (1024, 9), (12, 9)),
                                     ("spectral_conv2d_strips", 2, 5, 6, (512, 64), (12, 9)), ("spectral_conv1d_permode", 6, 5, 6, (256,), (121,)),
                                     ("spectral_conv1d_permode", 64, 20, 70, (256,), (100,))):
        per_mode = name.endswith("permode")
        x = torch.from_numpy(inputs.make_x(13, B, Ci, dims)).cuda()
        W = torch.from_numpy(inputs.make_W(13, Ci, Co * K[0] if per_mode else Co)).cuda()
        y = torch.zeros((B, Co) + dims, dtype=torch.complex64, device="cuda")
        layers.append((getattr(binding, name), x, W.reshape(Ci, Co, -1) if per_mode else W, y, () if per_mode else K))
    for _ in range(2):                                      # (the workspace reaches its largest size in the first round)
        for fn, x, W, y, K in layers:
            fn(x, W, y, *K)
    torch.cuda.synchronize()
    want = [y.clone() for _, _, _, y, _ in layers]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            for fn, x, W, y, K in layers:
                fn(x, W, y, *K)
    torch.cuda.current_stream().wait_stream(side)
    for _ in range(3):
        for _, _, _, y, _ in layers:
            y.zero_()
        layers[0][0](layers[0][1], layers[0][2], layers[0][3], *layers[0][4])
        layers[0][3].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for (_, _, _, y, _), w in zip(layers, want):
            assert torch.equal(torch.view_as_real(y), torch.view_as_real(w))


# real-valued layer (B, C_in, C_out, N, K): every N of the fused kernel, ragged channels, K = N/2
REAL_1D = [(4, 16, 16, 64, 16), (3, 5, 7, 64, 8), (2, 33, 40, 64, 32), (3, 9, 70, 128, 32), (2, 37, 17, 128, 64),
           (64, 64, 64, 256, 64), (5, 19, 130, 256, 32), (2, 40, 33, 256, 16), (3, 24, 96, 256, 128), (2, 17, 9, 512, 32),
           (2, 8, 40, 512, 256), (3, 13, 129, 1024, 128), (1, 1, 1, 1024, 64), (2, 20, 30, 1024, 32), (2, 16, 64, 1024, 256),
           (2, 128, 128, 1024, 128),
           # N = 1024 on the symmetric-wave kernel: whole blocks without the deep pipeline, K = 64 deep, and a mode
           # count between the built sizes (stays on the four-wave kernel, which masks bins)
           (2, 16, 128, 1024, 64), (2, 64, 256, 1024, 64), (2, 9, 11, 1024, 100),
           # enough workgroups for the symmetric-wave kernel by default (smaller batches run the four-wave kernel)
           (128, 16, 128, 1024, 64), (70, 9, 130, 1024, 128),
           # at most 64 outputs: the four-wave kernel whatever the batch; one more: the symmetric-wave kernel
           (130, 16, 64, 1024, 64), (130, 16, 65, 1024, 64)]


@pytest.mark.parametrize("shape", REAL_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_real_layer(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N, K = shape
    say(f"[case] spectral_conv1d_real {shape}")
    x = np.ascontiguousarray(inputs.make_x(900 + N + K, B, Ci, (N,)).real)          # float32, N(0, 1)
    W = inputs.make_W(900 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d_real(x, W, K)
    xd, Wd = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda()
    yd = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
    binding.spectral_conv1d_real(xd, Wd, yd, K)
    torch.cuda.synchronize()
    got = yd.cpu().numpy().astype(np.float64)
    rel = np.linalg.norm((got - want).ravel()) / np.linalg.norm(want.ravel())
    mx = np.max(np.abs(got - want)) / np.max(np.abs(want))
    say(f"   real: rel_l2={rel:.3e} max_abs/max|y|={mx:.3e}")
    assert rel <= REL_L2 and mx <= MAX_ABS


# mode counts between the built kernel sizes (the FNO literature uses 12, 20, 24, 48 ...): the kernels run the next
# built size and zero the surplus bins before the contraction.  (B, C_in, C_out, N, K)
ANY_K_1D = [(3, 5, 7, 64, 12), (2, 16, 40, 128, 20), (2, 33, 17, 256, 48), (3, 9, 70, 256, 100), (2, 8, 8, 256, 1),
            (2, 12, 20, 512, 40), (2, 24, 130, 1024, 24), (2, 32, 128, 1024, 100), (1, 3, 200, 256, 33), (2, 4, 4, 64, 5)]


@pytest.mark.parametrize("shape", ANY_K_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_1d_any_mode_count(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N, K = shape
    x = inputs.make_x(1000 + N + K, B, Ci, (N,))
    W = inputs.make_W(1000 + N + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    fns = ["spectral_conv1d", "spectral_conv1d_auto", "spectral_conv1d_staged"]
    if binding.workspace_bytes(1, 2, B, Ci, Co, N, K):
        fns.append("spectral_conv1d_pruned")
    if binding.workspace_bytes(1, 3, B, Ci, Co, N, K):
        fns += ["spectral_conv1d_fft_gemm", "spectral_conv1d_gemm_ifft"]
    for fn in fns:
        say(f"[case] {fn} {shape}")
        check(run_gpu(gpu, fn, x, W, K), want, fn)
    if 2 * K <= N:
        xr = np.ascontiguousarray(x.real)
        wantr, _ = oracle_mod.spectral_conv1d_real(xr, W, K)
        yd = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
        binding.spectral_conv1d_real(torch.from_numpy(xr).cuda(), torch.from_numpy(W).cuda(), yd, K)
        torch.cuda.synchronize()
        got = yd.cpu().numpy().astype(np.float64)
        assert np.linalg.norm((got - wantr).ravel()) / np.linalg.norm(wantr.ravel()) <= REL_L2
        assert np.max(np.abs(got - wantr)) / np.max(np.abs(wantr)) <= MAX_ABS


# (B, C_in, C_out, N1, N2, K1, K2): few images on grids of the image kernels with rounded mode counts (the kernels themselves: IMAGES_2D), strip
# pipeline with a rounded last axis, long pencils
ANY_K_2D = [(2, 3, 5, 64, 64, 12, 12), (1, 5, 33, 128, 256, 20, 48), (2, 4, 3, 256, 128, 64, 33), (1, 2, 2, 64, 256, 1, 5),
            (2, 3, 4, 32, 256, 8, 40), (1, 2, 3, 512, 64, 100, 12)]


@pytest.mark.parametrize("shape", ANY_K_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_K%dx%d" % s)
def test_2d_any_mode_count(gpu, oracle_mod, shape):
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] spectral_conv2d_rect {shape}")
    x = inputs.make_x(1100 + N1 + K2, B, Ci, (N1, N2))
    W = inputs.make_W(1100 + N1 + K2, Ci, Co)
    want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
    check(run_gpu_rect(gpu, "spectral_conv2d_rect", x, W, K1, K2), want, "rect any K")


def test_long_pencils_any_mode_count(gpu, oracle_mod):
    for (B, Ci, Co, N, K) in [(2, 5, 7, 2048, 100), (1, 3, 4, 4096, 300), (2, 4, 4, 4096, 17)]:
        say(f"[case] long pencils any K {(B, Ci, Co, N, K)}")
        x = inputs.make_x(1200 + N + K, B, Ci, (N,))
        W = inputs.make_W(1200 + N + K, Ci, Co)
        want, _ = oracle_mod.spectral_conv1d(x, W, K)
        for fn in ("spectral_conv1d_pruned", "spectral_conv1d_auto"):
            check(run_gpu(gpu, fn, x, W, K), want, fn)


# the 2-D FNO layer on real fields (B, C_in, C_out, N1, N2, M1, M2): block sizes that are built sizes and others,
# every row length, M1 at its maximum
FNO_2D = [(2, 3, 5, 64, 64, 12, 12), (2, 4, 4, 64, 64, 8, 16), (1, 5, 9, 128, 128, 16, 16), (3, 2, 3, 256, 256, 32, 64),
          (2, 3, 2, 64, 256, 5, 40), (2, 6, 3, 256, 64, 20, 7), (1, 17, 33, 128, 64, 1, 1), (9, 2, 2, 64, 128, 32, 32),
          (2, 3, 3, 128, 256, 24, 20)]


@pytest.mark.parametrize("shape", FNO_2D, ids=lambda s: "B%d_Ci%d_Co%d_N%dx%d_M%dx%d" % s)
def test_fno2d_real_layer(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N1, N2, M1, M2 = shape
    say(f"[case] fno2d_real {shape}")
    x = np.ascontiguousarray(inputs.make_x(1300 + N1 + M2, B, Ci, (N1, N2)).real)
    W = np.ascontiguousarray(inputs.make_W(1300 + N1 + M2, Ci, Co * 2 * M1 * M2).reshape(Ci, Co, 2 * M1, M2))
    want, _ = oracle_mod.fno2d_real(x, W)
    yd = torch.full((B, Co, N1, N2), float("nan"), dtype=torch.float32, device="cuda")
    binding.fno2d_real(torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), yd)
    torch.cuda.synchronize()
    got = yd.cpu().numpy().astype(np.float64)
    rel = np.linalg.norm((got - want).ravel()) / np.linalg.norm(want.ravel())
    mx = np.max(np.abs(got - want)) / np.max(np.abs(want))
    say(f"   fno2d: rel_l2={rel:.3e} max_abs/max|y|={mx:.3e}")
    assert rel <= REL_L2 and mx <= MAX_ABS


# Row stage of real images: every number of lanes per row (N2 / 16) with every number of bins per column (K2 / 16), one mode,
# the last mode, and one to many images per batch; tensors that are aligned to 8 bytes only (16-byte accesses in the kernels).
@pytest.mark.parametrize("N1,N2", [(64, 64), (64, 128), (128, 256), (256, 64), (256, 256)])
def test_fno2d_rows_of_every_width(gpu, oracle_mod, N1, N2):
    torch, binding = gpu
    for M2 in [m for m in (1, 7, 8, 9, 16, 17, 32, 33, 64) if 2 * m <= N2]:    # (more than 32: rows that skip the patch on their way in)
        for shift in (0, 2):
            B, Ci, Co, M1 = 2, 3, 5, 5 + M2 % 4
            say(f"[case] fno2d rows {(N1, N2, M1, M2, shift)}")
            x = np.ascontiguousarray(inputs.make_x(1350 + N1 + M2, B, Ci, (N1, N2)).real)
            W = np.ascontiguousarray(inputs.make_W(1350 + N2 + M2, Ci, Co * 2 * M1 * M2).reshape(Ci, Co, 2 * M1, M2))
            want, _ = oracle_mod.fno2d_real(x, W)
            xd = torch.empty(x.size + 4, dtype=torch.float32, device="cuda")[shift:shift + x.size].view(B, Ci, N1, N2)
            xd.copy_(torch.from_numpy(x))
            whole = torch.full((want.size + 8,), float("nan"), dtype=torch.float32, device="cuda")
            yd = whole[shift:shift + want.size].view(B, Co, N1, N2)
            binding.fno2d_real(xd, torch.from_numpy(W).cuda(), yd)
            torch.cuda.synchronize()
            close(yd.cpu().numpy().astype(np.float64), want, ("fno2d rows", N1, N2, M1, M2, shift))
            assert bool(torch.isnan(whole[:shift]).all()) and bool(torch.isnan(whole[shift + want.size:]).all())


# Channel counts around the blocks of the per-mode FP32 kernel (16 with one result per thread, 8 with four; four waves share a
# result's blocks): below one block, one to five blocks, every remainder's halves, batches that leave the last workgroup ragged.
@pytest.mark.parametrize("B,Co,M", [(3, 5, 9), (5, 33, 57)], ids=["one", "four"])
def test_permode_channel_blocks(gpu, oracle_mod, B, Co, M):
    torch, binding = gpu
    for Ci in (1, 7, 8, 9, 15, 16, 17, 23, 24, 31, 32, 33, 47, 64, 65, 79, 130):
        say(f"[case] permode channel blocks {(B, Ci, Co, M)}")
        x = np.ascontiguousarray(inputs.make_x(1370 + Ci, B, Ci, (128,)).real)
        W = np.ascontiguousarray(inputs.make_W(1370 + Ci, Ci, Co * M).reshape(Ci, Co, M))
        want, _ = oracle_mod.fno1d_real(x, W)
        yd = torch.full((B, Co, 128), float("nan"), dtype=torch.float32, device="cuda")
        binding.fno1d_real(torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), yd)
        torch.cuda.synchronize()
        close(yd.cpu().numpy().astype(np.float64), want, ("permode channel blocks", B, Ci, Co, M))


# The same blocks through the 2-D layer, whose small contractions the FP32 kernel runs (those of small 1-D layers are in the inverse kernel).
@pytest.mark.parametrize("B,Co,K1,K2", [(3, 5, 3, 3), (5, 33, 3, 19)], ids=["one", "four"])
def test_permode_channel_blocks_2d(gpu, oracle_mod, B, Co, K1, K2):
    torch, binding = gpu
    for Ci in (1, 7, 8, 9, 15, 16, 17, 23, 31, 33, 47, 65, 79):
        say(f"[case] permode channel blocks, 2-D {(B, Ci, Co, K1, K2)}")
        x = inputs.make_x(1375 + Ci, B, Ci, (64, 64))
        W = np.ascontiguousarray(inputs.make_W(1375 + Ci, Ci, Co * K1 * K2).reshape(Ci, Co, K1, K2))
        want, _ = oracle_mod.spectral_conv2d_permode(x, W)
        yd = torch.full((B, Co, 64, 64), float("nan"), dtype=torch.complex64, device="cuda")
        binding.spectral_conv2d_permode(torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), yd)
        torch.cuda.synchronize()
        close(yd.cpu().numpy(), want, ("permode channel blocks, 2-D", B, Ci, Co, K1, K2))


# Small per-mode layers, contraction and inverse in one kernel: every length and mode count it is built for, real and complex; one and two results per
# lane, one and several rounds of them, one output per workgroup up to 16, a last workgroup with one output, channels around the blocks of
# 8 and 16 and a round of four of them; and the limits of the rule (20 MB of weights read, 768 workgroups).
@pytest.mark.parametrize("N,K", [(64, 9), (64, 32), (64, 40), (128, 7), (128, 32), (128, 63), (128, 100), (256, 16), (256, 20), (256, 64), (256, 128), (256, 200),
                                 (1024, 16), (1024, 64), (1024, 127)], ids=lambda v: str(v))
def test_small_permode_layers(gpu, oracle_mod, N, K):
    torch, binding = gpu
    for B, Ci, Co in ((1, 1, 1), (2, 8, 17), (3, 33, 5), (2, 65, 9), (70, 3, 17), (300, 2, 3)) + (((384, 3, 2), (385, 3, 2)) if N == 256 else ()):
        say(f"[case] small permode {(B, Ci, Co, N, K)}")
        x = inputs.make_x(1385 + Ci, B, Ci, (N,))
        W = np.ascontiguousarray(inputs.make_W(1385 + Ci, Ci, Co * K).reshape(Ci, Co, K))
        yd = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
        binding.spectral_conv1d_permode(torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), yd)
        close(yd.cpu().numpy(), oracle_mod.spectral_conv1d_permode(x, W)[0], ("small permode", B, Ci, Co, N, K))
        if 2 * K > N:
            continue
        xr = np.ascontiguousarray(x.real)
        yr = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
        binding.fno1d_real(torch.from_numpy(xr).cuda(), torch.from_numpy(W).cuda(), yr)
        close(yr.cpu().numpy().astype(np.float64), oracle_mod.fno1d_real(xr, W)[0], ("small fno1d", B, Ci, Co, N, K))


# the 1-D FNO layer on real fields (B, C_in, C_out, N, M)
FNO_1D = [(4, 16, 16, 64, 16), (3, 5, 7, 64, 12), (9, 33, 40, 128, 20), (17, 6, 18, 256, 128), (2, 20, 30, 1024, 64),
          (11, 13, 17, 1024, 100), (2, 3, 3, 128, 1), (8, 3, 2, 256, 33)]


@pytest.mark.parametrize("shape", FNO_1D, ids=lambda s: "B%d_Ci%d_Co%d_N%d_M%d" % s)
def test_fno1d_real_layer(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N, M = shape
    say(f"[case] fno1d_real {shape}")
    x = np.ascontiguousarray(inputs.make_x(1400 + N + M, B, Ci, (N,)).real)
    W = np.ascontiguousarray(inputs.make_W(1400 + N + M, Ci, Co * M).reshape(Ci, Co, M))
    want, _ = oracle_mod.fno1d_real(x, W)
    yd = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
    binding.fno1d_real(torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), yd)
    torch.cuda.synchronize()
    got = yd.cpu().numpy().astype(np.float64)
    rel = np.linalg.norm((got - want).ravel()) / np.linalg.norm(want.ravel())
    mx = np.max(np.abs(got - want)) / np.max(np.abs(want))
    say(f"   fno1d: rel_l2={rel:.3e} max_abs/max|y|={mx:.3e}")
    assert rel <= REL_L2 and mx <= MAX_ABS


def test_every_1d_shape_either_runs_or_is_reported_unsupported(gpu, oracle_mod):
    """Sweeps N and K over their whole range for every 1-D entry point: a call must end in TFNO_OK or
    TFNO_ERR_UNSUPPORTED (never a launch error from a shape the dispatch accepted but no kernel was built for), and
    what runs must match the oracle."""
    torch, binding = gpu
    B, Ci, Co = 2, 3, 2
    ran = 0
    for e in range(1, 13):
        N = 1 << e
        x = inputs.make_x(1600 + e, B, Ci, (N,))
        xd = torch.from_numpy(x).cuda()
        xr = np.ascontiguousarray(x.real)
        xrd = torch.from_numpy(xr).cuda()
        W = inputs.make_W(1600 + e, Ci, Co)
        Wd = torch.from_numpy(W).cuda()
        ks = sorted({k for k in (1, 2, 3, 5, 8, 12, 16, 24, 32, 48, 64, 100, 128, 200, 256, 300, 512, 1000, 1024, 2048, 4096,
                                 N // 2, N) if 1 <= k <= N})
        for K in ks:
            want = None
            for fn in ("spectral_conv1d", "spectral_conv1d_pruned", "spectral_conv1d_fft_gemm", "spectral_conv1d_gemm_ifft",
                       "spectral_conv1d_auto"):
                yd = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
                try:
                    getattr(binding, fn)(xd, Wd, yd, K)
                except binding.TfnoError as err:
                    assert err.status == binding.ERR_UNSUPPORTED, (fn, N, K, err.status)
                    assert fn != "spectral_conv1d_auto", (N, K)
                    continue
                torch.cuda.synchronize()
                if want is None:
                    want, _ = oracle_mod.spectral_conv1d(x, W, K)
                got = yd.cpu().numpy().astype(np.complex128)
                close(got, want, (fn, N, K))
                ran += 1
            if 2 * K <= N:
                Wm = np.ascontiguousarray(np.repeat(W[:, :, None], K, axis=2))
                Wmd = torch.from_numpy(Wm).cuda()
                wantr = None
                for fn, args in (("spectral_conv1d_real", (xrd, Wd)), ("fno1d_real", (xrd, Wmd))):
                    yd = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
                    try:
                        if fn == "fno1d_real":
                            binding.fno1d_real(*args, yd)
                        else:
                            binding.spectral_conv1d_real(*args, yd, K)
                    except binding.TfnoError as err:
                        assert err.status == binding.ERR_UNSUPPORTED, (fn, N, K, err.status)
                        continue
                    torch.cuda.synchronize()
                    if wantr is None:
                        wantr, _ = oracle_mod.spectral_conv1d_real(xr, W, K)     # equal matrices: the same operator
                    got = yd.cpu().numpy().astype(np.float64)
                    close(got, wantr, (fn, N, K))
                    ran += 1
    say(f"   {ran} (entry point, N, K) combinations ran and matched the oracle")
    assert ran > 400


def test_every_2d_shape_either_runs_or_is_reported_unsupported(gpu, oracle_mod):
    """The same sweep for the 2-D entry points over N1, N2 in {32 .. 512} and mode counts from 1 to N/2."""
    torch, binding = gpu
    B, Ci, Co = 1, 2, 2
    ran = 0
    for N1 in (32, 64, 128, 256, 512):
        for N2 in (32, 64, 128, 256, 512):
            x = inputs.make_x(1700 + N1 + 3 * N2, B, Ci, (N1, N2))
            xd = torch.from_numpy(x).cuda()
            xr = np.ascontiguousarray(x.real)
            xrd = torch.from_numpy(xr).cuda()
            W = inputs.make_W(1700 + N1, Ci, Co)
            Wd = torch.from_numpy(W).cuda()
            for (K1, K2) in sorted({(1, 1), (5, 12), (16, 16), (24, 40), (64, 64), (N1 // 2, N2 // 2), (12, N2 // 2)}):
                if K1 > N1 or K2 > N2:
                    continue
                want, _ = oracle_mod.spectral_conv2d_rect(x, W, K1, K2)
                Wm = np.broadcast_to(W[:, :, None, None], (Ci, Co, K1, K2)).copy()
                for fn, args in (("spectral_conv2d_rect", (xd, Wd)), ("spectral_conv2d_permode", (xd, torch.from_numpy(Wm).cuda()))):
                    yd = torch.full((B, Co, N1, N2), float("nan"), dtype=torch.complex64, device="cuda")
                    try:
                        if fn == "spectral_conv2d_rect":
                            binding.spectral_conv2d_rect(*args, yd, K1, K2)
                        else:
                            binding.spectral_conv2d_permode(*args, yd)
                    except binding.TfnoError as err:
                        assert err.status == binding.ERR_UNSUPPORTED, (fn, N1, N2, K1, K2, err.status)
                        continue
                    torch.cuda.synchronize()
                    got = yd.cpu().numpy().astype(np.complex128)
                    close(got, want, (fn, N1, N2, K1, K2))
                    ran += 1
                M1 = K1 // 2
                if M1 >= 1 and 2 * K2 <= N2:
                    Wf = np.ascontiguousarray(inputs.make_W(1700 + K1 + K2, Ci, Co * 2 * M1 * K2).reshape(Ci, Co, 2 * M1, K2))
                    yd = torch.full((B, Co, N1, N2), float("nan"), dtype=torch.float32, device="cuda")
                    try:
                        binding.fno2d_real(xrd, torch.from_numpy(Wf).cuda(), yd)
                    except binding.TfnoError as err:
                        assert err.status == binding.ERR_UNSUPPORTED, ("fno2d_real", N1, N2, M1, K2, err.status)
                        continue
                    torch.cuda.synchronize()
                    wantf, _ = oracle_mod.fno2d_real(xr, Wf)
                    got = yd.cpu().numpy().astype(np.float64)
                    close(got, wantf, ("fno2d", N1, N2, M1, K2))
                    ran += 1
    say(f"   {ran} (entry point, N1, N2, K1, K2) combinations ran and matched the oracle")
    assert ran > 150


def test_channel_count_sweep(gpu, oracle_mod):
    """Ragged and boundary channel counts (around every tile size of the kernels) on the main entry points."""
    torch, binding = gpu
    vals = [1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 127, 128, 129, 160, 255, 256, 257]
    rs = np.random.default_rng(77)
    pairs = [(int(rs.choice(vals)), int(rs.choice(vals))) for _ in range(20)] + [(1, 257), (257, 1), (129, 129)]
    for idx, (Ci, Co) in enumerate(pairs):
        N, K, B = (256, 64, 2) if idx % 3 else (1024, 128, 1)
        x = inputs.make_x(1800 + idx, B, Ci, (N,))
        W = inputs.make_W(1800 + idx, Ci, Co)
        want, _ = oracle_mod.spectral_conv1d(x, W, K)
        fns = ["spectral_conv1d", "spectral_conv1d_pruned", "spectral_conv1d_auto"]
        if N == 256:
            fns += ["spectral_conv1d_fft_gemm", "spectral_conv1d_gemm_ifft"]
        for fn in fns:
            got = run_gpu(gpu, fn, x, W, K).astype(np.complex128)
            close(got, want, (fn, Ci, Co, N))
        xr = np.ascontiguousarray(x.real)
        wantr, _ = oracle_mod.spectral_conv1d_real(xr, W, K)
        yd = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
        binding.spectral_conv1d_real(torch.from_numpy(xr).cuda(), torch.from_numpy(W).cuda(), yd, K)
        torch.cuda.synchronize()
        got = yd.cpu().numpy().astype(np.float64)
        close(got, wantr, ("real", Ci, Co, N))
        # 2-D: strips of few images or, with more than half of the rows retained, image kernels and mode CGEMM; per-mode contraction
        x2 = inputs.make_x(1900 + idx, 1, Ci, (64, 64))
        want2, _ = oracle_mod.spectral_conv2d_rect(x2, W, 33, 16)
        close(run_image_kernels(gpu, x2, W, 33, 16).astype(np.complex128), want2, ("2d images", Ci, Co))
        want2, _ = oracle_mod.spectral_conv2d(x2, W, 16)
        got = run_gpu(gpu, "spectral_conv2d", x2, W, 16).astype(np.complex128)
        close(got, want2, ("2d", Ci, Co))
        Wm = np.broadcast_to(W[:, :, None, None], (Ci, Co, 16, 16)).copy()
        yd = torch.full((1, Co, 64, 64), float("nan"), dtype=torch.complex64, device="cuda")
        binding.spectral_conv2d_permode(torch.from_numpy(x2).cuda(), torch.from_numpy(Wm).cuda(), yd)
        torch.cuda.synchronize()
        got = yd.cpu().numpy().astype(np.complex128)
        close(got, want2, ("2d permode", Ci, Co))
    say(f"   {len(pairs)} channel-count pairs on 9-10 layers each")


def test_batch_size_sweep(gpu, oracle_mod):
    """Odd and boundary batch sizes on the kernels that group pencils, tiles or images (pruned sweeps, two long
    pencils per sweep, mode tiles shared by batch elements, the batch groups of the per-mode contraction)."""
    torch, binding = gpu
    Ci, Co = 3, 5
    for B in (1, 2, 3, 5, 7, 8, 9, 15, 16, 17, 31, 33, 65):
        for (fn, N, K) in (("spectral_conv1d_pruned", 64, 16), ("spectral_conv1d_pruned", 256, 32),
                           ("spectral_conv1d_pruned", 2048, 128), ("spectral_conv1d_gemm_ifft", 128, 32),
                           ("spectral_conv1d", 64, 8)):
            x = inputs.make_x(2000 + B + N, B, Ci, (N,))
            W = inputs.make_W(2000 + B + N, Ci, Co)
            want, _ = oracle_mod.spectral_conv1d(x, W, K)
            got = run_gpu(gpu, fn, x, W, K).astype(np.complex128)
            close(got, want, (fn, B, N, K))
        for (N, K) in ((64, 16), (256, 12)):
            x = inputs.make_x(2100 + B + N, B, Ci, (N,))
            Wm = np.ascontiguousarray(inputs.make_W(2100 + B + N, Ci, Co * K).reshape(Ci, Co, K))
            want, _ = oracle_mod.spectral_conv1d_permode(x, Wm)
            yd = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
            binding.spectral_conv1d_permode(torch.from_numpy(x).cuda(), torch.from_numpy(Wm).cuda(), yd)
            torch.cuda.synchronize()
            got = yd.cpu().numpy().astype(np.complex128)
            close(got, want, ("permode", B, N, K))
            xr = np.ascontiguousarray(x.real)
            wantr, _ = oracle_mod.fno1d_real(xr, Wm)
            yr = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
            binding.fno1d_real(torch.from_numpy(xr).cuda(), torch.from_numpy(Wm).cuda(), yr)
            torch.cuda.synchronize()
            got = yr.cpu().numpy().astype(np.float64)
            close(got, wantr, ("fno1d", B, N, K))
        x2 = np.ascontiguousarray(inputs.make_x(2200 + B, B, Ci, (64, 64)).real)
        Wf = np.ascontiguousarray(inputs.make_W(2200 + B, Ci, Co * 24 * 12).reshape(Ci, Co, 24, 12))
        wantf, _ = oracle_mod.fno2d_real(x2, Wf)
        yf = torch.full((B, Co, 64, 64), float("nan"), dtype=torch.float32, device="cuda")
        binding.fno2d_real(torch.from_numpy(x2).cuda(), torch.from_numpy(Wf).cuda(), yf)
        torch.cuda.synchronize()
        got = yf.cpu().numpy().astype(np.float64)
        close(got, wantf, ("fno2d", B))


def test_wide_output_slabs_with_ragged_channels(gpu, oracle_mod):
    """Batches large enough that the fused kernel keeps its widest output slabs (small batches are given narrower
    ones to fill the chip), with channel counts that leave the last slab, the last 32-output tile and the last
    channel block partly empty."""
    for (B, Ci, Co, N, K) in [(140, 5, 70, 64, 16), (150, 9, 130, 128, 32), (140, 33, 40, 256, 64), (130, 20, 96, 512, 64),
                              (135, 7, 100, 256, 128), (132, 17, 33, 1024, 32), (140, 3, 129, 64, 64)]:
        say(f"[case] wide slabs {(B, Ci, Co, N, K)}")
        x = inputs.make_x(2300 + N + K, B, Ci, (N,))
        W = inputs.make_W(2300 + N + K, Ci, Co)
        want, _ = oracle_mod.spectral_conv1d(x, W, K)
        check(run_gpu(gpu, "spectral_conv1d", x, W, K), want, "fused, wide slabs")
        if 2 * K <= N:
            torch, binding = gpu
            xr = np.ascontiguousarray(x.real)
            wantr, _ = oracle_mod.spectral_conv1d_real(xr, W, K)
            yd = torch.full((B, Co, N), float("nan"), dtype=torch.float32, device="cuda")
            binding.spectral_conv1d_real(torch.from_numpy(xr).cuda(), torch.from_numpy(W).cuda(), yd, K)
            torch.cuda.synchronize()
            got = yd.cpu().numpy().astype(np.float64)
            close(got, wantr, "real layer")


# N = 256 has three more fused kernels behind the dispatch: the single-operand-tile kernel (K = 128, more batch rows
# than CUs; two workgroups per CU), the eight-wave kernel (256 outputs per workgroup for C_out > 128, and 32 or 64 for
# batches of at most 256 workgroups) and the two-group kernel (C_out > 128: 256 outputs per workgroup).  Shapes that reach each of them with whole and ragged channel blocks, absent output slabs and mode counts
# between the built sizes.  (B, C_in, C_out, N, K)
N256_SPECIAL = [
    (300, 5, 70, 256, 128),      # single tile, masked, 128-output slab partly empty
    (260, 20, 33, 256, 100),     # single tile, masked, 64-output slab, K rounded up to 128
    (257, 9, 30, 256, 128),      # single tile, masked, 32-output slab
    (258, 16, 64, 256, 128),     # single tile, whole blocks
    # (the 256-output kernels take over from 192 batch rows on)
    (193, 64, 256, 256, 48),     # two-group kernel, K rounded up to 64
    (192, 64, 160, 256, 64),     # two-group kernel, three of eight output slabs absent
    (200, 96, 192, 256, 32),     # two-group kernel, six 16-channel blocks
    (192, 128, 256, 256, 128),   # eight-wave kernel, whole blocks
    (195, 70, 200, 256, 128),    # eight-wave kernel, masked
    (200, 48, 136, 256, 32),     # eight-wave kernel (48 channels are not whole 32-channel blocks), masked
    (191, 64, 256, 256, 64),     # one row short of the rule: the four-wave kernel, two 128-output slabs per row
    # at most 256 workgroups of 32 (K <= 64: or 64) outputs: eight waves with those slabs
    (64, 20, 33, 256, 64),       # 32-output slabs, masked, the second slab holds one channel
    (8, 64, 256, 256, 128),      # 32-output slabs, exactly 256 workgroups, whole blocks
    (100, 33, 100, 256, 48),     # 64-output slabs (400 workgroups of 32 outputs would be too many), K rounded up
    (256, 8, 64, 256, 32),       # 64-output slabs, exactly 256 workgroups
    (257, 5, 64, 256, 32),       # one row more: the four-wave kernel
    (150, 33, 100, 256, 64),     # 300 workgroups of 64 outputs: the four-wave kernel
    (100, 7, 100, 256, 128),     # K = 128 has no 64-output eight-wave kernel: the four-wave kernel
    # N = 128, K = 64 with more batch rows than CUs: the single-operand-tile kernel (two workgroups per CU)
    (300, 20, 70, 128, 64), (260, 32, 33, 128, 50), (258, 64, 128, 128, 64), (257, 5, 9, 128, 64),
    (300, 16, 200, 128, 64),     # ... two slabs per row; the dispatch keeps the fused kernel here
    (300, 16, 200, 128, 32),     # ... and takes the CGEMM + iFFT variant at K = 32
    # N = 128, K <= 32, 33 .. 64 outputs, more than two batch rows per CU: single operand tile, the partial sums of the
    # split contraction added in turns into one epilogue tile (three workgroups per CU)
    (600, 20, 40, 128, 32), (520, 32, 64, 128, 32), (513, 5, 40, 128, 16), (600, 64, 33, 128, 20), (530, 32, 64, 128, 16),
    (512, 32, 64, 128, 32),      # one row short of the rule: the double-buffered kernel
    (600, 32, 32, 128, 32),      # 32 outputs: the double-buffered kernel, four partial sums side by side
    # ... and the same form with four output tiles: N = 128 (whole channel blocks only), N = 64 (any channel count)
    (520, 32, 128, 128, 32), (513, 64, 256, 128, 16), (520, 32, 130, 128, 32), (520, 20, 128, 128, 32),
    (600, 32, 128, 64, 16), (520, 20, 96, 64, 32), (513, 9, 70, 64, 8), (512, 32, 128, 64, 16),
    # N = 64, at most 32 outputs, more than three batch rows per CU: single operand tile, four workgroups per CU;
    # N = 128 likewise for a single half-empty block of input channels
    (800, 32, 32, 64, 16), (770, 16, 20, 64, 32), (769, 5, 9, 64, 8), (768, 32, 32, 64, 16),
    (600, 16, 16, 128, 32), (520, 9, 30, 128, 16), (600, 17, 16, 128, 32),
    # N = 256, K <= 64, more than four batch rows per CU, whole channel blocks: single operand tile, three workgroups per CU
    (1025, 16, 32, 256, 32), (1100, 32, 64, 256, 64), (1030, 16, 128, 256, 32), (1026, 32, 64, 256, 20),
    (1030, 16, 128, 256, 64),    # K = 64 with 128 outputs would spill there: the double-buffered kernel
    (1030, 24, 64, 256, 32),     # 24 channels are not whole blocks: the double-buffered kernel
]


@pytest.mark.parametrize("shape", N256_SPECIAL, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_n256_dispatched_kernels(gpu, oracle_mod, shape):
    B, Ci, Co, N, K = shape
    say(f"[case] N = 256 dispatch {shape}")
    x = inputs.make_x(2400 + Ci + K, B, Ci, (N,))
    W = inputs.make_W(2400 + Ci + K, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d", x, W, K), want, "fused")
    check(run_gpu(gpu, "spectral_conv1d_auto", x, W, K), want, "auto")


def test_round_trip_identity_and_determinism(gpu):
    """K = N, W = I gives y = x; two runs give bitwise equal output."""
    torch, binding = gpu
    N, C = 256, 48
    x = inputs.make_x(3, 4, C, (N,))
    W = np.eye(C, dtype=np.complex64)
    a = run_gpu(gpu, "spectral_conv1d", x, W, N)
    b = run_gpu(gpu, "spectral_conv1d", x, W, N)
    assert np.array_equal(a.view(np.float32), b.view(np.float32))
    check(a, x.astype(np.complex128), "round trip")


def test_empty_batch_and_error_paths(gpu):
    torch, binding = gpu
    x = torch.zeros((0, 4, 64), dtype=torch.complex64, device="cuda")
    W = torch.zeros((4, 4), dtype=torch.complex64, device="cuda")
    y = torch.zeros((0, 4, 64), dtype=torch.complex64, device="cuda")
    binding.spectral_conv1d(x, W, y, 16)
    binding.spectral_conv1d_staged(x, W, y, 16)
    x = torch.zeros((1, 4, 64), dtype=torch.complex64, device="cuda")
    with pytest.raises(binding.TfnoError) as e:
        binding.spectral_conv1d(x, W, x, 16)           # y aliases x
    assert e.value.status == binding.ERR_ALIAS
    y = torch.zeros((1, 4, 64), dtype=torch.complex64, device="cuda")
    with pytest.raises(binding.TfnoError) as e:
        binding.spectral_conv1d(x, W, y, 65)
    assert e.value.status == binding.ERR_SHAPE
    torch.cuda.synchronize()


# Scaling the input or the weights by a power of two only changes exponents, so every entry point must return the
# scaled result bit for bit: the transforms multiply by twiddles and add, and the contraction splits each operand into
# three BF16 terms whose exponent range is that of float32.  A split that lost low-order terms to underflow, or a
# path that mixed scaled and unscaled quantities, would show here.
@pytest.mark.parametrize("entry,shape", [("spectral_conv1d", (3, 24, 40, 1024, 128)), ("spectral_conv1d", (5, 32, 64, 256, 128)),
                                         ("spectral_conv1d", (4, 64, 256, 256, 64)), ("spectral_conv1d_pruned", (3, 70, 65, 256, 64)),
                                         ("spectral_conv2d", (2, 8, 8, 64, 16)), ("spectral_conv2d", (2, 9, 1, 64, 16)), ("spectral_conv2d", (1, 4, 3, 512, 40)),
                                         ("spectral_conv1d_auto", (3, 24, 40, 1024, 50)), ("spectral_conv1d_auto", (3, 24, 40, 1000, 50)), ("spectral_conv1d_auto", (9, 5, 40, 39, 20)),
                                         ("spectral_conv2d_staged", (2, 8, 8, 85, 12)),
                                         ("spectral_conv1d_permode", (16, 24, 33, 256, 100)), ("spectral_conv1d_permode", (64, 40, 64, 256, 100)),
                                         ("spectral_conv1d_permode", (3, 20, 7, 64, 12))],
                         ids=lambda v: v if isinstance(v, str) else "x".join(map(str, v)))
def test_power_of_two_scaling_is_exact(gpu, entry, shape):
    torch, binding = gpu
    B, Ci, Co, N, K = shape
    say(f"[case] scaling {entry} {shape}")
    dims = (N, N) if "2d" in entry else (N,)
    x = inputs.make_x(4242, B, Ci, dims)
    per_mode = entry.endswith("permode")
    W = inputs.make_W(4242, Ci, Co * K if per_mode else Co)

    def run(x, W):
        if not per_mode:
            return run_gpu(gpu, entry, x, W, K)
        y = torch.full((B, Co, N), float("nan"), dtype=torch.complex64, device="cuda")
        getattr(binding, entry)(torch.from_numpy(x).cuda(), torch.from_numpy(W.reshape(Ci, Co, K)).cuda(), y)
        return y.cpu().numpy()

    base = run(x, W)
    assert np.isfinite(base.view(np.float32)).all()
    for ex, ew in ((30, 0), (-30, 0), (0, 25), (-20, -20), (40, -45)):
        got = run(x * np.float32(2.0 ** ex), W * np.float32(2.0 ** ew))
        want = base * np.float32(2.0 ** (ex + ew))
        assert np.array_equal(got.view(np.float32), want.view(np.float32)), (entry, shape, ex, ew)


def test_workspace_growth_does_not_disturb_earlier_work_on_another_stream(gpu, oracle_mod):
    """A call that uses the workspace is enqueued on a side stream behind a long queue of other launches; a call
    with a larger workspace need follows on the default stream at once.  The binding synchronises the device before
    it replaces the registered buffer, so the first call still finds its intermediates: its result must match the
    oracle."""
    torch, binding = gpu
    binding.set_workspace(None)                               # start from no workspace at all
    xa = inputs.make_x(2500, 6, 24, (256,)); Wa = inputs.make_W(2500, 24, 40)
    xb = inputs.make_x(2501, 24, 48, (256,)); Wb = inputs.make_W(2501, 48, 64)
    xad, Wad = torch.from_numpy(xa).cuda(), torch.from_numpy(Wa).cuda()
    xbd, Wbd = torch.from_numpy(xb).cuda(), torch.from_numpy(Wb).cuda()
    ya = torch.full((6, 40, 256), float("nan"), dtype=torch.complex64, device="cuda")
    yb = torch.full((24, 64, 256), float("nan"), dtype=torch.complex64, device="cuda")
    filler = torch.empty(1 << 26, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(20):
            filler.fill_(1.0)                                 # keeps the side stream busy ahead of the call
        binding.spectral_conv1d_pruned(xad, Wad, ya, 64, stream=side.cuda_stream)
    binding.spectral_conv1d_pruned(xbd, Wbd, yb, 64)          # needs a larger workspace
    torch.cuda.synchronize()
    check(ya.cpu().numpy(), oracle_mod.spectral_conv1d(xa, Wa, 64)[0], "first call (side stream)")
    check(yb.cpu().numpy(), oracle_mod.spectral_conv1d(xb, Wb, 64)[0], "second call (larger workspace)")


# ----------------------------------------------------- full benchmark sizes, every batch element

def full_size_inputs(torch, w):
    Wn = inputs.make_W(w.seed, w.C_in, w.C_out)
    xd = torch.empty((w.B, w.C_in) + w.spatial, dtype=torch.complex64, device="cuda")
    for b in range(w.B):
        xd[b] = torch.from_numpy(inputs.make_x_element(w.seed, b, w.C_in, w.spatial)).cuda()
    return xd, Wn, torch.from_numpy(Wn).cuda()


def full_size_run(gpu, w, fn_name, xd, Wd):
    """The whole workload in the launch configuration the benchmark times; the output starts as NaN."""
    torch, binding = gpu
    yd = torch.full((w.B, w.C_out) + w.spatial, float("nan"), dtype=torch.complex64, device="cuda")
    getattr(binding, fn_name)(xd, Wd, yd, w.K)
    torch.cuda.synchronize()
    assert not torch.isnan(torch.view_as_real(yd)).any().item(), f"{fn_name}: some outputs were never written"
    return yd


def whole_batch_against_oracle(gpu, oracle_mod, w, fn_name, xd, Wn, yd, chunk=16):
    """Every batch element of the full-size output against the oracle, `chunk` elements at a time (the float64 result
    of the 2-D configuration would not fit comfortably at once): the tolerance must hold for every chunk and the
    relative L2 error for every single batch element (each is one workgroup row or one group of images on the GPU,
    so a fault tied to a compute unit, an XCD residue or a grid slab shows up in its own element)."""
    say(f"[case] {fn_name} {w.name}: all {w.B} batch elements against the oracle")
    worst = 0.0
    for b0 in range(0, w.B, chunk):
        b1 = min(w.B, b0 + chunk)
        xb = xd[b0:b1].cpu().numpy()
        want, _ = oracle_fn(oracle_mod, w.dims)(xb, Wn, w.K)
        got = yd[b0:b1].cpu().numpy().astype(np.complex128)
        close(got, want, f"{fn_name} {w.name} b={b0}..{b1 - 1}")
        err = np.linalg.norm((got - want).reshape(b1 - b0, -1), axis=1) / np.linalg.norm(want.reshape(b1 - b0, -1), axis=1)
        assert err.max() <= REL_L2, (fn_name, w.name, b0 + int(err.argmax()), float(err.max()))
        worst = max(worst, float(err.max()))
    say(f"   worst batch element: rel_l2={worst:.3e}")


def whole_batch_against_reference(gpu, oracle_mod, w, fn_name, xd, Wn, yd, y_ref, sample_b):
    """A variant's full-size output: every batch row against the fused kernel's output on the device (which
    whole_batch_against_oracle has tied to the oracle; two float32 paths agree to a few rounding errors), and the
    batch elements `sample_b` against the oracle itself."""
    torch, _ = gpu
    say(f"[case] {fn_name} {w.name}: all rows against the fused output, b={sample_b} against the oracle")
    d = torch.view_as_real(yd - y_ref).reshape(w.B, -1).double().norm(dim=1)
    r = torch.view_as_real(y_ref).reshape(w.B, -1).double().norm(dim=1)
    rel = (d / r).max().item()
    say(f"   worst row against the fused output: rel_l2={rel:.3e}")
    assert rel <= 5e-6, (fn_name, w.name, rel)
    for b in sample_b:
        want, _ = oracle_fn(oracle_mod, w.dims)(xd[b:b + 1].cpu().numpy(), Wn, w.K)
        check(yd[b].cpu().numpy()[None], want, f"{fn_name} {w.name} b={b}")


def full_size_config(gpu, oracle_mod, w, fused_fn, others):
    torch, _ = gpu
    xd, Wn, Wd = full_size_inputs(torch, w)
    y_ref = full_size_run(gpu, w, fused_fn, xd, Wd)
    whole_batch_against_oracle(gpu, oracle_mod, w, fused_fn, xd, Wn, y_ref)
    # E|y|^2 = 4 (K/N)^dims for these input distributions: a property that holds at any size
    e2 = torch.mean(torch.abs(y_ref.view(-1)[: 1 << 24]) ** 2).item()
    assert abs(e2 / (4 * (w.K / w.N) ** w.dims) - 1) < 0.05
    for fn_name, sample_b in others:
        yd = full_size_run(gpu, w, fn_name, xd, Wd)
        whole_batch_against_reference(gpu, oracle_mod, w, fn_name, xd, Wn, yd, y_ref, sample_b)
        del yd
    del xd, y_ref
    torch.cuda.empty_cache()


def test_config3_full_size(gpu, oracle_mod):
    full_size_config(gpu, oracle_mod, inputs.CONFIGS[2], "spectral_conv1d",
                     [("spectral_conv1d_staged", [0, 255]), ("spectral_conv1d_pruned", [101]), ("spectral_conv1d_auto", [7])])


def test_config4_full_size(gpu, oracle_mod):
    full_size_config(gpu, oracle_mod, inputs.CONFIGS[3], "spectral_conv2d", [("spectral_conv2d_staged", [0, 31])])


@pytest.mark.parametrize("w", inputs.sweep_configs(), ids=lambda w: w.name)
def test_config5_sweep_full_size(gpu, oracle_mod, w):
    full_size_config(gpu, oracle_mod, w, "spectral_conv1d",
                     [("spectral_conv1d_auto", [0, 511]), ("spectral_conv1d_staged", [257]), ("spectral_conv1d_pruned", [3]),
                      ("spectral_conv1d_fft_gemm", [509]), ("spectral_conv1d_gemm_ifft", [2, 508])])


SYM_1D = [(2, 32, 128, 1024, 128),   # two blocks of loads in flight (even block count >= 4), no masks
          (1, 48, 256, 1024, 64),
          (2, 16, 128, 1024, 128),   # unmasked, two blocks only
          (3, 13, 129, 1024, 128),   # masked
          (1, 1, 1, 1024, 64)]


@pytest.mark.parametrize("kernel", ["ws", "generic", "sym"])
def test_alternative_n1024_kernels_in_a_child_process(gpu, oracle_mod, tmp_path, kernel):
    """N = 1024 runs the symmetric-wave kernel by default when the grid fills half the chip (K in {64, 128}) and the
    four-wave kernel below that; TFNO_KERNEL (read once per process) selects the wave-specialised kernel (ws), the
    four-wave kernel (generic) or the symmetric-wave kernel (sym) for every batch size.  The real-valued layer follows
    the same switch."""
    import os
    import subprocess
    import textwrap
    say(f"[case] TFNO_KERNEL={kernel} child process")
    out = str(tmp_path / f"{kernel}.npz")
    code = textwrap.dedent(f"""
        import numpy as np, torch
        from paper_2504_11681_amd import binding, inputs
        res = {{}}
        for i, (B, Ci, Co, N, K) in enumerate({SYM_1D!r}):
            x = inputs.make_x(40 + i, B, Ci, (N,)); W = inputs.make_W(40 + i, Ci, Co)
            y = torch.empty((B, Co, N), dtype=torch.complex64, device='cuda')
            binding.spectral_conv1d(torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda(), y, K)
            torch.cuda.synchronize()
            res['y%d' % i] = y.cpu().numpy()
            if K <= N // 2:
                yr = torch.empty((B, Co, N), dtype=torch.float32, device='cuda')
                binding.spectral_conv1d_real(torch.from_numpy(np.ascontiguousarray(x.real)).cuda(), torch.from_numpy(W).cuda(), yr, K)
                torch.cuda.synchronize()
                res['r%d' % i] = yr.cpu().numpy()
        np.savez({out!r}, **res)
    """)
    env = dict(os.environ, TFNO_KERNEL=kernel)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    subprocess.run([sys.executable, "-c", code], check=True, env=env, cwd=root, timeout=110)
    got = np.load(out)
    for i, (B, Ci, Co, N, K) in enumerate(SYM_1D):
        x = inputs.make_x(40 + i, B, Ci, (N,)); W = inputs.make_W(40 + i, Ci, Co)
        check(got["y%d" % i], oracle_mod.spectral_conv1d(x, W, K)[0], f"{kernel} {(B, Ci, Co, N, K)}")
        wantr = oracle_mod.spectral_conv1d_real(np.ascontiguousarray(x.real), W, K)[0]
        gotr = got["r%d" % i].astype(np.float64)
        assert np.linalg.norm((gotr - wantr).ravel()) <= 1e-5 * np.linalg.norm(wantr.ravel()), (kernel, "real", i)
        assert np.abs(gotr - wantr).max() <= 1e-4 * np.abs(wantr).max(), (kernel, "real", i)


def test_fp32_contraction_kernels_in_a_child_process(gpu, oracle_mod, tmp_path):
    """TFNO_CONTRACTION=f32 (read once per process) selects the FP32-MFMA contraction kernels: the generic fused
    1-D kernel for N = 1024 and the FP32 mode CGEMM of the 2-D path.  A child process runs both and saves the
    results; they are compared with the oracle here."""
    import os
    import subprocess
    import textwrap
    say("[case] TFNO_CONTRACTION=f32 child process")
    out = str(tmp_path / "f32.npz")
    code = textwrap.dedent(f"""
        import numpy as np, torch
        from paper_2504_11681_amd import binding, inputs
        x1 = inputs.make_x(31, 2, 20, (1024,)); W1 = inputs.make_W(31, 20, 40)
        y1 = torch.empty((2, 40, 1024), dtype=torch.complex64, device='cuda')
        binding.spectral_conv1d(torch.from_numpy(x1).cuda(), torch.from_numpy(W1).cuda(), y1, 128)
        x2 = inputs.make_x(32, 2, 5, (128, 128)); W2 = inputs.make_W(32, 5, 70)
        y2 = torch.empty((2, 70, 128, 128), dtype=torch.complex64, device='cuda')
        binding.spectral_conv2d(torch.from_numpy(x2).cuda(), torch.from_numpy(W2).cuda(), y2, 32)
        torch.cuda.synchronize()
        np.savez({out!r}, y1=y1.cpu().numpy(), y2=y2.cpu().numpy())
    """)
    env = dict(os.environ, TFNO_CONTRACTION="f32")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    subprocess.run([sys.executable, "-c", code], check=True, env=env, cwd=root, timeout=110)
    got = np.load(out)
    x1 = inputs.make_x(31, 2, 20, (1024,)); W1 = inputs.make_W(31, 20, 40)
    check(got["y1"], oracle_mod.spectral_conv1d(x1, W1, 128)[0], "f32 1-D N=1024")
    x2 = inputs.make_x(32, 2, 5, (128, 128)); W2 = inputs.make_W(32, 5, 70)
    check(got["y2"], oracle_mod.spectral_conv2d(x2, W2, 32)[0], "f32 2-D 128x128")


# (entry, sizes): the direct-sum transforms (long and short lengths, several pencils to a workgroup, columns of a grid), the
# per-mode contraction with 8 x 8, 4 x 4 and fewer results per thread
F32_LAYERS = [("staged1d", 2, 3, 4, 421, 50), ("staged1d", 3, 20, 9, 1000, 33), ("staged1d", 1, 2, 2, 4095, 100), ("staged1d", 7, 5, 6, 39, 39),
              # (of these two the first does not fit the workspace with the matrix transform, the second just does)
              ("grid2d", 1, 64, 1, 83, 97, 4, 97), ("grid2d", 1, 64, 1, 83, 97, 4, 90), ("staged1d", 1, 3, 4, 127, 127), ("staged1d", 1, 3, 4, 63, 63),
              ("grid2d", 2, 3, 4, 85, 48, 12, 20), ("grid2d", 2, 2, 3, 48, 85, 48, 9), ("grid2d", 1, 3, 2, 421, 12, 30, 12),
              ("permode1d", 128, 9, 128, 256, 256), ("permode1d", 100, 8, 100, 256, 128), ("permode1d", 60, 20, 70, 256, 100), ("permode1d", 6, 33, 7, 1024, 60),
              ("permode1d", 128, 24, 128, 256, 64), ("permode1d", 128, 16, 129, 256, 64), ("permode1d", 64, 31, 100, 128, 50), ("permode1d", 64, 32, 128, 256, 60), ("permode1d", 64, 64, 64, 256, 73)]


def f32_layer(torch, binding, layer):
    """One layer of F32_LAYERS on the GPU: x, W, y as arrays."""
    entry, B, Ci, Co, *dims = layer
    n = len(dims) // 2
    space, K = tuple(dims[:n]), dims[n:]
    x = inputs.make_x(1700 + space[0], B, Ci, space)
    W = inputs.make_W(1700 + space[0], Ci, Co * K[0] if entry == "permode1d" else Co)
    if entry == "permode1d":
        W = W.reshape(Ci, Co, K[0])
    xd, Wd = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda()
    yd = torch.full((B, Co) + space, float("nan"), dtype=torch.complex64, device="cuda")
    if entry == "permode1d":
        binding.spectral_conv1d_permode(xd, Wd, yd)
    elif entry == "staged1d":
        binding.spectral_conv1d_staged(xd, Wd, yd, K[0])
    else:
        binding.spectral_conv2d_rect_staged(xd, Wd, yd, *K)
    torch.cuda.synchronize()
    return x, W, yd.cpu().numpy()


def test_fp32_general_layers_in_a_child_process(gpu, oracle_mod, tmp_path):
    """TFNO_CONTRACTION=f32: lengths with odd factors by direct sums, the per-mode contraction on its FP32 kernel.  By default the
    direct sums run where whole tiles of spectra and the half-transformed fields do not fit the workspace (same bits).  Per-mode
    layers run that kernel by default as well below 294912 results (393216 below 32 channels) or 16 channels, outputs or
    batch elements (same bits); the others run on the matrix pipe, with the error of the FP32 sums (which depends on the results
    per thread) or less, also with few channels: leaving out the smallest products would make it 4 % more at 16 of them."""
    import os
    import subprocess
    import textwrap
    torch, binding = gpu
    say("[case] TFNO_CONTRACTION=f32 child process, general layers")
    out = str(tmp_path / "f32_general.npz")
    code = textwrap.dedent(f"""
        import sys
        sys.path.insert(0, "tests")
        import numpy as np, torch
        from paper_2504_11681_amd import binding
        from test_parity_gpu import F32_LAYERS, f32_layer
        np.savez({out!r}, *[f32_layer(torch, binding, layer)[2] for layer in F32_LAYERS])
    """)
    env = dict(os.environ, TFNO_CONTRACTION="f32")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    subprocess.run([sys.executable, "-c", code], check=True, env=env, cwd=root, timeout=110)
    got = np.load(out)
    for i, layer in enumerate(F32_LAYERS):
        entry, B, Ci, Co, *dims = layer
        x, W, default = f32_layer(torch, binding, layer)
        y = got["arr_%d" % i]
        if entry == "permode1d":
            N, K = dims
            f = np.exp(-2j * np.pi * np.outer(np.arange(N), np.arange(K)) / N)
            X = x.astype(np.complex128) @ f
            want = np.matmul(X.transpose(2, 0, 1), W.astype(np.complex128).transpose(2, 0, 1)).transpose(1, 2, 0) @ np.conj(f.T) / N
            same = np.array_equal(y.view(np.float32), default.view(np.float32))
            matrix_pipe = B >= 16 and Co >= 16 and Ci >= 16 and B * K * Co >= (393216 if Ci < 32 else 294912)
            assert same != matrix_pipe, (layer, same)
            errs = [np.linalg.norm(v - want) / np.linalg.norm(want) for v in (default, y)]
            say(f"   default {errs[0]:.3e}, FP32 {errs[1]:.3e}")
            assert not matrix_pipe or K > 64 or Ci >= 32 or errs[0] <= 1.03 * errs[1], layer
        else:
            N1, N2, K1, K2 = dims if entry == "grid2d" else (1, dims[0], 1, dims[1])
            if N2 & (N2 - 1):                             # (powers of two: K2 may be rounded up)
                need = -(-B * K1 * K2 // 128) * 128 * (Ci + Co) + (B * N1 * K2 * max(Ci, Co) if N1 > 1 else 0)
                fits = need <= B * (Ci + Co) * (N1 * N2 + K1 * K2)
                assert np.array_equal(y.view(np.float32), default.view(np.float32)) != fits, (layer, fits)
            want = (oracle_mod.spectral_conv1d if entry == "staged1d" else oracle_mod.spectral_conv2d_rect)(x, W, *dims[len(dims) // 2:])[0]
        check(y, want, f"f32 {layer}")


# Column kernels on both sides of the rules by which an XCD takes neighbouring columns: truncated spectra of more than 16 columns from 256
# workgroups on (258, 520 and 260 of them, 258 and 260 not shared evenly by the eight XCDs, and 24), whole fields from 403 MB on (200 fields of
# 512 x 512 points, 419 MB, and 104, 218 MB; their workgroups are always a multiple of eight); against float64 sums over the kept modes.
@pytest.mark.parametrize("shape", [(43, 3, 3, 64, 90, 9, 20), (65, 2, 1, 128, 300, 10, 50), (3, 2, 1, 128, 300, 10, 50), (13, 8, 1, 512, 512, 3, 5),
                                   (25, 8, 1, 512, 512, 3, 5)],
                         ids=lambda s: "B%d_%d_%d_%dx%d_K%dx%d" % s)
def test_column_kernels_with_neighbouring_columns(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N1, N2, K1, K2 = shape
    say(f"[case] columns {shape}")
    x = torch.view_as_complex(torch.randn(B, Ci, N1, N2, 2, generator=torch.Generator().manual_seed(N1 + N2)))
    W = torch.from_numpy(inputs.make_W(1390 + N1, Ci, Co))
    y = torch.full((B, Co, N1, N2), float("nan"), dtype=torch.complex64, device="cuda")
    call = binding.spectral_conv2d_rect if N2 % 16 == 0 and not N2 & (N2 - 1) else binding.spectral_conv2d_rect_staged
    call(x.cuda(), W.cuda(), y, K1, K2)
    torch.cuda.synchronize()
    f1 = np.exp(-2j * np.pi * np.outer(np.arange(K1), np.arange(N1)) / N1)
    f2 = np.exp(-2j * np.pi * np.outer(np.arange(N2), np.arange(K2)) / N2)
    X = f1 @ (x.numpy().astype(np.complex128) @ f2)                             # [B, Ci, K1, K2]
    Y = np.tensordot(X, W.numpy().astype(np.complex128), axes=([1], [0]))       # [B, K1, K2, Co]
    want = f1.conj().T @ np.moveaxis(Y, -1, 1) @ f2.conj().T / (N1 * N2)
    close(y.cpu().numpy().astype(np.complex128), want, ("columns", shape))


# The 256-output kernel: one block of 32 channels, whole blocks, a ragged last one, ragged outputs.
@pytest.mark.parametrize("Ci,Co", [(1, 129), (32, 256), (33, 160), (70, 250), (256, 256)])
def test_channel_blocks_of_the_256_output_kernel(gpu, oracle_mod, Ci, Co):
    B, N, K = 200, 256, 128
    x, W = inputs.make_x(2400 + Ci, B, Ci, (N,)), inputs.make_W(2400 + Ci, Ci, Co)
    say(f"[case] channel blocks {(B, Ci, Co, N, K)}")
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d", x, W, K), want, "256-output kernel")


# Fused 1-D kernels with four and more blocks of channels, the last one ragged, and more workgroups than the eight XCDs hold at a
# time: a batch whose rows are all equal gives the same bits in every row, and different rows agree with the oracle.
# (B, C_in, C_out, N, K)
MANY_BLOCKS = [
    (300, 130, 130, 128, 64), (300, 70, 70, 256, 128), (400, 50, 70, 256, 100), (520, 130, 70, 64, 16),     # single operand tile, 128 outputs
    (140, 70, 100, 256, 64), (140, 70, 100, 512, 64), (132, 41, 100, 1024, 32), (300, 33, 45, 1024, 64),    # double-buffered
    (200, 100, 250, 256, 128), (200, 256, 256, 256, 128), (200, 70, 200, 256, 64),                          # 256 outputs
]


@pytest.mark.parametrize("shape", MANY_BLOCKS, ids=lambda s: "B%d_Ci%d_Co%d_N%d_K%d" % s)
def test_equal_rows_give_equal_bits(gpu, oracle_mod, shape):
    torch, binding = gpu
    B, Ci, Co, N, K = shape
    say(f"[case] equal rows {shape}")
    x, W = inputs.make_x(2450 + Ci, B, Ci, (N,)), inputs.make_W(2450 + Ci, Ci, Co)
    want, _ = oracle_mod.spectral_conv1d(x, W, K)
    check(run_gpu(gpu, "spectral_conv1d", x, W, K), want, "different rows")
    row = torch.from_numpy(x[7:8]).cuda()
    y = torch.empty((B, Co, N), dtype=torch.complex64, device="cuda")
    binding.spectral_conv1d(row.expand(B, Ci, N).contiguous(), torch.from_numpy(W).cuda(), y, K)
    torch.cuda.synchronize()
    close(y[0].cpu().numpy().astype(np.complex128), want[7], ("equal rows", shape))
    bits = torch.view_as_real(y).view(torch.int32)
    assert bool((bits == bits[:1]).all()), "rows differ"
