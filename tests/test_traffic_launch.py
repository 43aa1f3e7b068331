"""The bytes that the fused filter's launches have to move: the matrix, U and W in every
step, the filtered block in steps 5, 8, ... and the last one (a model of its own, beside
Eq. 2 with five block rows in every step)."""
import pytest

from paper_1803_02156_amd import traffic

N, NNZ = 1000, 12987


@pytest.mark.parametrize("prec,s", [(0, 16), (1, 8)])
@pytest.mark.parametrize("n_b", [1, 32])
def test_launch_bytes_are_three_launches_averaged(prec, s, n_b):
    block, matrix = N * n_b * s, NNZ * (s + 4)
    r, w = traffic.launch_bytes(N, NNZ, n_b, prec)
    assert 3 * r == pytest.approx(3 * matrix + 7 * block, rel=1e-15)     # U, W three times, X once
    assert 3 * w == pytest.approx(4 * block, rel=1e-15)                  # W three times, X once
    r2, w2 = traffic.step_bytes(N, NNZ, n_b, prec)
    assert r + w == pytest.approx(r2 + w2 - 4 / 3 * block, rel=1e-15)    # Eq. 2 moves X in every step


@pytest.mark.parametrize("prec,s", [(0, 16), (1, 8)])
@pytest.mark.parametrize("n_p,updates", [(2, 0), (3, 1), (4, 1), (5, 1), (6, 2), (8, 2), (9, 3), (100, 33)])
def test_needed_filter_bytes_step_by_step(prec, s, n_p, updates):
    n_b, blocks = 8, 3
    block, matrix = N * n_b * s, NNZ * (s + 4)
    total, done = sum(traffic.start_bytes(N, NNZ, n_b, prec)), 0
    for p in range(3, n_p + 1):
        total += matrix + 3 * block
        if (p - 3) % 3 == 2 or p == n_p:
            total, done = total + 2 * block, done + 1
    assert done == updates
    assert traffic.needed_filter_bytes(N, NNZ, n_b * blocks, n_b, n_p, prec) == blocks * total
    assert traffic.needed_filter_bytes(N, NNZ, n_b, n_b, n_p, prec) <= traffic.filter_bytes(N, NNZ, n_b, n_b, n_p, prec)
