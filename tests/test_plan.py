"""The launch choices of csrc/plan.h, which are pure functions of sizes and compute units: compiled here with the host
compiler and called at sizes on both sides of where one shape was measured faster than the other. No choice changes a
result, so the parity tests cannot see a wrong one."""

import pytest

from plan_shim import K1, K3, PPO, norm_fused, response_blocks, stream_shape

# on the 256 compute units of an MI355X, which the calls below take by default


@pytest.mark.parametrize("term", [K1, K3, PPO])
@pytest.mark.parametrize("n", [513, 1024, 8192, 20000, 1 << 22])
@pytest.mark.parametrize("mean", [100, 550, 1100, 6000, 16384])
def test_many_responses_take_one_block(term, n, mean):
    """More than two responses per CU: four blocks of threads each were 1.3 to 4 times slower at every length."""
    assert response_blocks(term, n * mean, n) == 1


@pytest.mark.parametrize("term,n,mean,want", [
    (K3, 64, 512, 1), (K3, 256, 1300, 1), (K3, 256, 1600, 4), (K3, 1, 16384, 4),
    (K3, 257, 4096, 1), (K3, 512, 6000, 4),
    (K1, 256, 2048, 1), (K1, 256, 3072, 4), (K1, 512, 6000, 1), (K1, 512, 8192, 4),
    (PPO, 256, 1024, 1), (PPO, 200, 1300, 4), (PPO, 64, 1600, 4), (PPO, 512, 6000, 1), (PPO, 257, 8192, 4),
])
def test_long_responses_take_four_blocks_where_they_pay(term, n, mean, want):
    assert response_blocks(term, n * mean, n) == want


@pytest.mark.parametrize("rows,d,V", [
    # few halves per CU: the lone wave was up to 1.9 times slower
    (1, 1536, 1000), (1, 2048, 1000), (16, 4096, 1000), (16, 8192, 1000), (1, 1024, 8000), (1, 5120, 2000),
    (17, 512, 8000), (17, 1024, 8000), (32, 2048, 8000), (32, 4096, 8000), (32, 7168, 1000),
    (33, 128, 1000), (48, 256, 8000), (64, 512, 32000), (64, 1024, 8000), (64, 4096, 16000), (64, 8192, 1000),
    # a second half on some CUs
    (64, 4096, 50257), (33, 1024, 40000), (64, 1024, 80000), (16, 512, 50257),
    # rows a power of two apart
    (17, 2048, 90000), (32, 2048, 196608), (32, 4096, 165000), (64, 2048, 151936), (64, 4096, 80000),
    (1, 8192, 50257), (16, 8192, 151936), (16, 4096, 196608), (1, 6144, 165000), (17, 1024, 90000), (17, 16384, 50257), (64, 8192, 196608),
    # not all resident, and more rows than it takes
    (1, 4096, 200000), (65, 4096, 151936),
])
def test_decode_stays_on_two_wave_tiles(rows, d, V):
    assert stream_shape(rows, d, V) is None


@pytest.mark.parametrize("rows,d,V,want", [
    (5, 2048, 151936, (1, 2)), (5, 2048, 57000, (1, 8)), (1, 2048, 32000, (1, 8)), (16, 4096, 151936, (1, 4)),
    (16, 4096, 32000, (1, 8)), (1, 5120, 8000, (1, 8)), (1, 128, 1000, (1, 8)), (16, 1024, 32000, (1, 8)),
    (20, 3584, 151936, (2, 8)), (32, 4096, 32000, (2, 8)), (32, 4096, 50257, (2, 8)), (32, 4096, 65536, (2, 4)),
    (32, 4096, 151936, (2, 4)), (25, 2048, 151936, (2, 4)), (25, 2048, 50257, (2, 8)),
    (64, 5120, 152064, (4, 8)), (64, 4096, 151936, (4, 8)), (64, 2560, 32000, (4, 8)), (1, 8192, 32000, (1, 4)),
    (64, 7168, 24000, (4, 8)), (17, 12288, 12000, (2, 8)), (1, 2048, 72000, (1, 8)), (5, 2048, 196608, (1, 2)),
])
def test_decode_takes_a_wave_per_half(rows, d, V, want):
    assert stream_shape(rows, d, V) == want


@pytest.mark.parametrize("d,T,fused", [
    (4096, 65536, True), (4096, 72000, False), (4096, 90000, False), (4096, 100000, False), (4096, 110000, True),
    (4096, 120000, True), (4096, 131071, True), (4096, 131072, True), (4096, 138564, True), (4096, 1 << 23, True),
    (2048, 65536, True), (2048, 90000, False), (2048, 110000, True), (2048, 131072, True), (2048, 140000, False),
    (2048, 170000, True), (2048, 196608, True), (2048, 200000, False), (2048, 230000, True), (2048, 262143, True),
    (2048, 262144, True), (2048, 300000, True),
])
def test_norm_backward_sums_in_the_grad_x_pass(d, T, fused):
    """One workgroup per block of rows, where the blocks fill the CUs that have the most of them: 5-15% faster there,
    up to 20% slower elsewhere."""
    assert norm_fused(T, d) is fused
