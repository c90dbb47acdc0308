"""Which kernel a linear on codes runs (csrc/qift_route.h), on the CPU: sizes whose kernels were timed, and every
kernel's limits over a grid of sizes."""
import pytest

from route_probe import ask

# (W4, N, K, M, workspace, us of the kernels that take it): sizes on both sides of each line of the rule
MEASURED = [
    # more rows than one round of batch workgroups
    (0, 40960, 4096, 33, 0, {"batch": 34.89, "gemm": 20.28, "skinny": 33.77}),
    (0, 40960, 20480, 33, 1, {"batch": 125.15, "gemm_split": 66.53, "gemm": 86.06}),
    (1, 40960, 4096, 48, 0, {"batch": 43.26, "gemm": 28.46, "skinny": 52.72}),
    (1, 40960, 2048, 17, 0, {"batch": 22.32, "skinny": 14.56}),
    # wide, short K
    (0, 16384, 2048, 17, 0, {"batch": 8.38, "skinny": 5.94}),
    (0, 28672, 2048, 24, 0, {"batch": 10.25, "skinny": 9.08}),
    (1, 28672, 2048, 20, 0, {"batch": 13.11, "skinny": 10.66}),
    (0, 16384, 1024, 48, 0, {"batch": 7.84, "gemm": 8.32, "skinny": 7.24}),
    (1, 16384, 1024, 33, 0, {"batch": 7.47, "gemm": 9.62, "skinny": 7.47}),
    # long K with the skinny split
    (0, 1000, 14336, 17, 1, {"batch": 11.12, "skinny": 12.23, "skinny_split": 8.92}),
    (0, 1000, 14336, 32, 1, {"batch": 11.54, "skinny": 16.67, "skinny_split": 9.60}),
    (0, 2048, 14336, 16, 1, {"batch": 9.67, "skinny_split": 8.30, "decode": 13.67}),
    (0, 2048, 11008, 20, 1, {"batch": 9.32, "skinny": 11.52, "skinny_split": 8.73}),
    (0, 4096, 14336, 24, 1, {"batch": 14.11, "skinny": 15.56, "skinny_split": 12.41}),
    (0, 1000, 14336, 33, 1, {"batch": 11.27, "skinny_split": 10.21}),
    (0, 300, 16384, 40, 1, {"batch": 11.61, "skinny_split": 10.44}),
    (0, 4096, 11008, 16, 1, {"batch": 8.36, "skinny_split": 9.36, "decode": 11.47}),
    # just past 4096 k, few rows
    (0, 300, 5120, 12, 0, {"batch": 6.08, "codes": 5.58}),
    (0, 1000, 5120, 17, 0, {"batch": 7.72, "skinny": 6.62}),
    (1, 300, 4096, 15, 0, {"batch": 5.74, "codes": 5.05}),
    (1, 4096, 5120, 15, 0, {"batch": 7.66, "codes": 7.19}),
    # W4, long K, 17 to 27 tokens
    (1, 3072, 11008, 20, 0, {"batch": 15.13, "skinny": 13.52}),
    (1, 4096, 11008, 17, 0, {"batch": 15.22, "skinny": 13.45}),
    # very long K with the split GEMM
    (1, 4096, 16384, 33, 1, {"batch": 18.50, "gemm_split": 16.98, "skinny": 26.32}),
    (1, 12288, 20480, 40, 1, {"batch": 49.87, "gemm_split": 42.38, "gemm": 115.40}),
    (0, 12288, 20480, 33, 1, {"batch": 35.24, "gemm_split": 30.55, "gemm": 82.17}),
    (0, 28672, 20480, 48, 1, {"batch": 67.40, "gemm_split": 56.18, "gemm": 84.44}),
    (0, 22016, 11008, 33, 1, {"batch": 34.29, "gemm_split": 31.76, "gemm": 46.42}),
    (1, 28672, 14336, 33, 1, {"batch": 64.34, "gemm_split": 57.68, "gemm": 77.25}),
    # W4 rows just past a round of the batch kernel's tiles, with the split GEMM
    (1, 5120, 13824, 33, 1, {"batch": 20.71, "gemm_split": 16.89}),
    (1, 9000, 7168, 26, 1, {"batch": 17.77, "gemm_split": 16.31}),
    (0, 8192, 28672, 52, 1, {"batch": 36.11, "gemm_split": 33.32}),
    (0, 70000, 4096, 30, 0, {"batch": 40.01, "skinny": 45.05}),
    (1, 2560, 9728, 21, 0, {"batch": 12.74, "skinny": 11.75}),
    (1, 777, 6208, 32, 0, {"batch": 8.59, "skinny": 7.93}),
    (0, 777, 6208, 13, 0, {"batch": 5.94, "codes": 6.99}),
    # what the batch kernel and the GEMM keep
    (0, 4096, 4096, 24, 0, {"batch": 6.27, "skinny": 6.59}),
    (0, 6144, 4096, 9, 0, {"batch": 5.63, "codes": 6.59}),
    (1, 12288, 4096, 48, 0, {"batch": 13.26, "gemm": 25.14, "skinny": 22.02}),
    (0, 22016, 4096, 64, 1, {"batch": 16.58, "gemm_split": 23.65, "gemm": 19.31, "skinny": 28.12}),
    (0, 28672, 4096, 64, 1, {"batch": 20.22, "gemm_split": 25.55, "gemm": 19.88, "skinny": 28.72}),
    (1, 22016, 4096, 40, 1, {"batch": 19.79, "gemm_split": 24.46, "gemm": 25.54, "skinny": 30.20}),
    (0, 4096, 14336, 64, 1, {"batch": 14.47, "gemm_split": 16.48, "gemm": 52.63, "skinny": 30.35}),
    (1, 28672, 4096, 16, 0, {"batch": 20.33, "codes": 22.99}),
    (0, 16384, 8192, 9, 0, {"batch": 13.41, "codes": 24.05}),
]


@pytest.mark.parametrize("w4,N,K,M,ws,us", MEASURED, ids=[f"{'w4' if c[0] else 'w2'}-{c[1]}x{c[2]}-m{c[3]}" for c in MEASURED])
def test_route_takes_the_faster_kernel(w4, N, K, M, ws, us):
    kernel, *_ = ask([(w4, N, K, M, "codes" in us, ws)])[0]
    # 4 %: twice what repeated timings of one kernel differed by
    assert us[kernel] <= 1.04 * min(us.values()), (kernel, us)


def test_route_stays_within_the_kernels_limits():
    Ns = [1, 16, 63, 300, 1000, 2048, 4095, 4096, 4097, 8192, 8193, 12288, 16383, 16384, 16385, 24576, 24577, 32768, 32769, 70000]
    Ks = [64, 256, 1088, 2048, 3072, 4096, 4160, 8128, 8192, 8256, 11008, 12288, 14336, 16384, 16448, 20480, 65536]
    Ms = [1, 4, 5, 8, 9, 12, 16, 17, 23, 24, 27, 28, 32, 33, 47, 48, 64, 65, 200, 2048]
    qs = [(w4, N, K, M, c, ws) for w4 in (0, 1) for N in Ns for K in Ks for M in Ms
          for c in ((0, 1) if M <= 16 and K <= 16384 else (0,)) for ws in (0, 1)]
    for (w4, N, K, M, codes, ws), (kernel, gemm_ranges, skinny_ranges, _) in zip(qs, ask(qs)):
        q = (w4, N, K, M, codes, ws, kernel)
        if kernel == "batch":
            assert 5 <= M <= 64, q
        elif kernel == "gemm_split":
            assert ws and gemm_ranges >= 2, q
        elif kernel == "gemm":
            assert M > 16, q
        elif kernel == "skinny":
            # up to 32 tokens W2 of at most four units a slice, beyond two (the instances there are)
            assert 16 < M <= 64 and K <= (4096 if M > 32 else 16384 if w4 else 8192), q
        elif kernel == "skinny_split":
            assert ws and not w4 and M <= 47 and K <= 16384 and skinny_ranges >= 2 and not (M <= 16 and codes), q
        elif kernel == "codes":
            assert codes and M <= 16, q
        else:
            assert M <= 16 and not codes, q


# (W4, N, K, M, us of the tiled GEMM with tiles of 64, 96 and 128 tokens, us of its split over K)
TILES = [
    (0, 9000, 7168, 900, {64: 74.03, 96: 63.95, 128: 76.18}, None),
    (0, 9000, 20480, 1024, {64: 204.58, 96: 177.59, 128: 217.2}, None),
    (0, 12288, 14336, 800, {64: 141.46, 96: 125.85, 128: 150.15}, None),
    (0, 28672, 20480, 300, {64: 207.1, 96: 176.6, 128: 213.33}, None),
    (0, 5120, 14336, 2048, {64: 140.04, 96: 126.37, 128: 150.24}, None),
    (0, 3072, 2048, 1024, {64: 13.77, 96: 16.43, 128: 18.8}, 25.32),
    (0, 16384, 2048, 150, {64: 12.64, 96: 15.14, 128: 17.58}, 20.87),
    (0, 700, 2944, 90, {64: 16.25}, 11.11),
    (0, 1000, 4096, 128, {64: 17.92, 96: 21.61, 128: 26.58}, 12.32),
    (0, 4096, 4096, 256, {64: 17.97, 96: 21.96, 128: 26.33}, 15.66),
    (0, 3072, 5120, 150, {64: 21.88, 96: 27.08, 128: 32.01}, 15.81),
    (0, 12288, 5120, 300, {64: 23.94, 96: 28.51, 128: 32.84}, 33.89),
    (0, 12288, 7168, 300, {64: 29.73, 96: 35.3, 128: 41.61}, 39.15),
    (0, 9000, 7168, 65, {64: 29.03}, 21.89),
    (0, 12288, 8192, 256, {64: 31.43, 96: 37.66, 128: 45.63}, 40.94),
    (0, 4096, 8192, 700, {64: 30.71, 96: 36.9, 128: 45.13}, 40.61),
    (0, 9000, 11008, 192, {64: 40.25, 96: 50.0, 128: 60.44}, 33.1),
    (0, 6144, 14336, 450, {64: 51.22, 96: 62.64, 128: 75.59}, 58.61),
    (0, 1000, 20480, 1900, {64: 72.17, 96: 88.13, 128: 108.42}, 49.69),
    (1, 9000, 4096, 65, {64: 22.38, 96: 25.23, 128: 26.9}, 19.68),
    (1, 5120, 5120, 150, {64: 28.22, 96: 31.49, 128: 37.41}, 23.64),
    (1, 4096, 5120, 300, {64: 27.45, 96: 31.29, 128: 37.21}, 24.28),
    (1, 5120, 7168, 65, {64: 34.13, 96: 39.51, 128: 44.86}, 23.13),
    (1, 16384, 8192, 128, {64: 47.32, 96: 53.99, 128: 57.04}, 41.68),
    (1, 12288, 14336, 150, {64: 71.14, 96: 88.47, 128: 92.1}, 61.36),
    (1, 6144, 20480, 400, {64: 101.91, 96: 119.9, 128: 129.88}, 83.23),
]


@pytest.mark.parametrize("w4,N,K,M,us,split", TILES, ids=[f"{'w4' if c[0] else 'w2'}-{c[1]}x{c[2]}-m{c[3]}" for c in TILES])
def test_gemm_tiles_and_split(w4, N, K, M, us, split):
    (plain, *_), (kernel, _, _, tokens) = ask([(w4, N, K, M, 0, 0), (w4, N, K, M, 0, 1)])
    assert plain == "gemm" and us[tokens] <= 1.04 * min(us.values()), (tokens, us)
    if split is not None:
        assert kernel == ("gemm_split" if split < us[tokens] else "gemm"), (kernel, us[tokens], split)
