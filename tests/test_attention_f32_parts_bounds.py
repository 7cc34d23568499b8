"""The arithmetic of fp32 attention on two fp16 parts per number, on the CPU: powers of two from the first tile of 32 keys, parts, and the conditions
under which a workgroup keeps its result (otherwise it works on fp32 products).  Products and sums are exact here, so that the error is
that of the parts alone: wherever the conditions hold, it has to be no more than what the formula gives in plain fp32."""
import numpy as np
import pytest

SCALE_LOG2 = np.log2(np.e) / np.sqrt(128)
P = 2.0 ** 11   # what weights are scaled by


def _power(largest, top, of_zero=32.0):
    """The power of two that takes `largest` to [2^top, 2^(top + 1))."""
    e = np.frexp(np.where(largest == 0, 1, largest))[1] - 1
    return np.where(largest == 0, of_zero, np.exp2(top - e))


def _parts(x):
    """fp16 parts of scaled numbers, as float64."""
    first = x.astype(np.float16).astype(np.float64)
    return first, (x - first).astype(np.float16).astype(np.float64)


def _product(a, b):   # a @ b.T without the product of the second parts
    (a1, a2), (b1, b2) = _parts(a), _parts(b)
    return a1 @ b1.T + a1 @ b2.T + a2 @ b1.T


def parts_attention(Q, K, V):
    """O, log2-sum-exp2 and whether the result is kept, for queries [N_q][128] over keys and values [N][128] (float32)."""
    Q, K, V = [x.astype(np.float64) for x in (Q, K, V)]
    q_up, k_up = _power(np.abs(Q).max(1, keepdims=True), 14, 2.0 ** 40), _power(np.abs(K[:32]).max(), 10)
    v_up = _power(np.abs(V[:32]).max(0), 10)
    with np.errstate(over="ignore", invalid="ignore"):
        to_log2 = SCALE_LOG2 / (q_up * k_up)
        s = _product(Q * q_up, K * k_up) * to_log2
        m = s.max(1, keepdims=True)
        p = np.exp2(s - m)
        l = p.sum(1, keepdims=True)
        o = _product(p * P, (V * v_up).T)                     # scaled and not divided by l
        lse = m + np.log2(l)
    k_seen, v_seen = np.abs(K * k_up).max(), np.abs(V * v_up).max(0)
    kept = k_seen < 65504 and v_seen.max() < 65504
    # logits: half a step, 2^-25, of each of 128 numbers of a key times the query's, which are below 2^15, and the other way round, below 2^16
    kept &= (to_log2 <= 2.0 ** -15).all()
    # values and weights: every query over the features,
    N, down = len(K), np.where(v_seen == 0, 0, 1 / (P * v_up))
    least = np.maximum((v_seen * down).max() * P * max(2.0 ** -12, N * 2.0 ** -19), (64 * l * down).max(1))
    kept &= (np.abs(o * down).max(1) >= least).all()
    # and over four queries every feature that has four adjacent keys with values of less than 2^-11 of the first tile's (fewer: 2^-20), not all 0
    quads = np.abs(np.pad(V * v_up, ((0, -N % 4), (0, 0)))).reshape(-1, 4, 128).max(1)
    quads[N // 4:] *= 2.0 ** 9
    mixed = ((quads > 0) & (quads < 0.5)).any(0)
    kept &= (np.abs(o).reshape(-1, 4, 128).max(1) >= np.maximum(v_seen * P * 2.0 ** -14, 16 * l).reshape(-1, 4, 128).max(1))[:, mixed].all()
    return o / (P * v_up) / l, lse, kept


def exact_attention(Q, K, V):
    Q, K, V = [x.astype(np.float64) for x in (Q, K, V)]
    s = Q @ K.T * SCALE_LOG2
    m = s.max(1, keepdims=True)
    p = np.exp2(s - m)
    return p @ V / p.sum(1, keepdims=True), m + np.log2(p.sum(1, keepdims=True))


def fp32_attention(Q, K, V):
    s = Q @ K.T * np.float32(SCALE_LOG2)
    m = s.max(1, keepdims=True)
    p = np.exp2(s - m)
    return p @ V / p.sum(1, keepdims=True), m + np.log2(p.sum(1, keepdims=True))


def errors(result, exact, V):
    """Largest relative error of a query's row (2-norm), of a number against the size of its feature's values (their lower quartile), largest
    error of the log-sum-exp."""
    (o, lse), (ref, ref_lse) = result, exact
    by_row = np.linalg.norm(o - ref, axis=1) / np.linalg.norm(ref, axis=1)
    by_feature = np.abs(o - ref).max(0) / np.quantile(np.abs(V), 0.25, axis=0)
    return np.array([by_row.max(), by_feature.max(), np.abs(lse - ref_lse).max()])


def _inputs(N, seed=3):
    g = np.random.default_rng(seed)
    return [g.standard_normal((n, 128)).astype(np.float32) for n in (64, N, N)]


def _without_weight(Q, K, rows, b=600):   # e^-53
    Q[:, 0], K[:, 0] = 1, 0
    K[rows, 0] = -b


def case_normal(x, Q, K, V):
    Q *= x
    return 1e-2 <= x <= 3


def case_masked_key(x, Q, K, V):        # a key of the first tile at -x
    _without_weight(Q, K, 5, x)
    return x <= 1e3


def case_query_channel(x, Q, K, V):     # a channel of the queries that no key uses
    Q[:, 7], K[:, 7] = x, 0
    return x <= 1e2


def case_zeros_then_small(x, Q, K, V):  # a first tile of zeros, products of the same size as ever behind it
    K[:32] = 0
    K[32:] /= x
    Q *= x
    return x == 1


def case_large_value(x, Q, K, V):       # one row of values without weight
    _without_weight(Q, K, 5)
    V[5] = x
    return x <= 10


def case_large_values_in_a_tile(x, Q, K, V):
    _without_weight(Q, K, slice(0, 32))
    V[:32] *= x
    return x <= 10


def case_one_feature(x, Q, K, V):       # of small values, but for a row without weight
    _without_weight(Q, K, 5)
    V[:, 9] *= 1e-4
    V[5, 9] = x * 1e-4
    return x <= 10


def case_sink(x, Q, K, V):              # a key without values that takes all but 1 / x of the weight
    Q[:, 0], K[:, 0] = 16, 0
    K[3], V[3] = 0, 0
    K[3, 0] = np.float16(np.log(x) / np.sqrt(2))   # (its logit is one product, exact in parts: see below)
    return x <= 3


def case_one_key(x, Q, K, V):           # all queries see one key, some of whose values are next to 0
    Q[:, 0], K[:, 0] = 10, 0
    K[7, 0] = 40
    V *= x
    V[7, ::3] *= 1e-4
    return True


def case_uniform(x, Q, K, V):           # the same weights everywhere, values that nearly cancel
    Q[:] = 0
    V[:, ::5] -= V[:, ::5].mean(0)
    V *= x
    return True


CASES = [case_normal, case_masked_key, case_query_channel, case_zeros_then_small, case_large_value, case_large_values_in_a_tile, case_one_feature, case_sink,
         case_one_key, case_uniform]


@pytest.mark.parametrize("N", [20, 52, 320])
@pytest.mark.parametrize("case", CASES, ids=lambda f: f.__name__[5:])
def test_kept_results_are_as_good_as_fp32(case, N):
    kept_ones = 0
    for x in 10.0 ** np.arange(-2, 15, 0.5):
        if x < 1 and case is not case_normal:
            continue
        Q, K, V = _inputs(N)
        ordinary = case(x, Q, K, V)
        *result, kept = parts_attention(Q, K, V)
        assert kept or not ordinary, f"{x}: ordinary inputs would go to fp32 products"
        if kept:   # (twice fp32's error or its error on N(0, 1); a number may be ten times its feature's quartile)
            kept_ones += 1
            exact = exact_attention(Q, K, V)
            assert (errors(result, exact, V) <= [2, 4, 2] * np.maximum(errors(fp32_attention(Q, K, V), exact, V), 5e-7)).all(), x
    assert kept_ones > 0


def test_a_logit_of_one_product():
    """Where roundings do not average: up to 2^-21 off, of which 2^-22 is the product of the second parts (fp32: 2^-24)."""
    g = np.random.default_rng(2)
    q, k = g.uniform(0.25, 32, (2, 1 << 18)).astype(np.float32).astype(np.float64)
    (q1, q2), (k1, k2) = _parts(q * 1024), _parts(k * 1024)
    off = np.abs((q1 * k1 + q1 * k2 + q2 * k1) / (q * k * 2.0 ** 20) - 1)
    assert 2.0 ** -23 < off.max() <= 2.0 ** -21


def test_without_the_conditions():
    """What they are there for: the parts alone lose a masked key's neighbours."""
    Q, K, V = _inputs(320)
    case_masked_key(1e12, Q, K, V)
    o, _, kept = parts_attention(Q, K, V)
    ref, _ = exact_attention(Q, K, V)
    assert not kept and np.linalg.norm(o - ref) > 0.5 * np.linalg.norm(ref)


def test_parts_are_within_2_to_the_minus_23():
    g = np.random.default_rng(1)
    x = g.uniform(0.25, 65504, 1 << 20) * np.exp2(-g.integers(0, 10, 1 << 20).astype(np.float64))
    x = np.maximum(x, 0.25).astype(np.float32).astype(np.float64)
    first, second = _parts(x)
    assert (np.abs(x - first - second) <= 2.0 ** -23 * x).all()   # down to 1/4; below, half a step of the second part's
    y = (g.uniform(0, 0.25, 1 << 20)).astype(np.float32).astype(np.float64)
    first, second = _parts(y)
    assert (np.abs(y - first - second) <= 2.0 ** -25).all()
