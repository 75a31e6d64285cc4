"""The launch rule of the few-row kernel (host code): the calls of the tests reach every instance and every count of K shares that it
takes, and the lines of the dense rule lie where the tests look."""
import random

import pytest

import few_rows as fr


@pytest.mark.parametrize("family,shape,K,N,E,top,step,host", fr.CASES)
def test_cases_take_the_shape_they_name(family, shape, K, N, E, top, step, host):
    assert fr.grouped_shape(family, K, N, fr.counts(E, top, step), host) == shape


@pytest.mark.parametrize("family", list(fr.FORMATS))
def test_no_call_takes_a_shape_without_a_case(family):
    named = {c[1] for c in fr.CASES if c[0] == family}
    rng = random.Random(17)

    def log(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    for _ in range(3000):
        E, top = log(1, 256), log(1, 64)
        rows = [top] + [rng.randint(0, top) if rng.random() < 0.7 else 0 for _ in range(E - 1)]
        K, N = 64 * log(2, 448), log(1, 28672)   # (of one group there is no mix)
        shape = fr.grouped_shape(family, K, N, rows, rng.random() < 0.6)
        assert shape in named, (K, N, E, top)
        assert fr.dense_shape(family, K, N, rng.randint(2, 32))[0] in named


@pytest.mark.parametrize("family,K,N,M,taken", fr.DENSE)
def test_dense_lines(family, K, N, M, taken):
    assert fr.dense_shape(family, K, N, M)[1] == taken
