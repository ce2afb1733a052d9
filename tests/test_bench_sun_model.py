"""The SU(N) work model of the benchmark, product by product (CPU only)."""

import pytest

import bench


@pytest.mark.parametrize("N,operands,products", [
    (2, "permutes", 14), (3, "permutes", 15), (4, "permutes", 18), (6, "permutes", 18),
    (2, "lds", 18), (5, "lds", 18), (8, "lds", 18),
    (4, "matrix cores", 16.5), (7, "matrix cores", 16.5), (8, "matrix cores", 16.5)])
def test_products_of_a_link_and_stage(N, operands, products):
    assert bench.sun_products(N, operands) == products
    # four links, three stages; 8 N^3 flop a product, 64 N^2 beside them
    assert bench.sun_flops_per_site_step(N, operands) == 12 * (products * 8 * N ** 3 + 64 * N * N)


def test_matrix_core_products_of_a_site():
    upper, lower, us, exp, update = 6 * 3, 12 * 2, 4, 4 * 4, 4
    assert 4 * bench.sun_products(8, "matrix cores") == upper + lower + us + exp + update
