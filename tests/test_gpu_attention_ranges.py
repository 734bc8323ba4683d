"""Prefill attention where scores and values span large ranges, against the CPU oracle: one layer whose queries have one
large component, on caches whose keys answer it with an offset chosen position by position."""
import numpy as np
import pytest

import workloads as W
from oracle import decoder as O
from tests import _util as U

pytestmark = pytest.mark.gpu

# 24 query heads: one sequence makes a grid of at most 128 tiles, six of them a larger one (different kernels over long
# key ranges)
STEEP = {d: W.DecoderShape("steep%d" % d, L=1, H=512, Hq=24, Hkv=12, d=d, F=256, rope_base=10000.0, seed=40 + d) for d in (64, 128)}


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _bits(x):
    return W.bf16_bits_from_f32(np.asarray(x, dtype=np.float32))


def _layer(s):
    """Seeded weights, but every query head's component of the lowest rotary frequency is 4 times the first (normalised)
    hidden value, and its rotation partner zero."""
    bits = dict(W.layer_weights_bits(s, 0))
    wq = bits["wq"].copy()
    for h in range(s.Hq):
        wq[h * s.d + s.d // 2 - 1] = 0
        wq[h * s.d + s.d - 1] = 0
        wq[h * s.d + s.d // 2 - 1, 0] = _bits([4.0])[0]
    bits["wq"] = wq
    return bits


def _hidden(s, T, step):
    """Hidden values N(0, 1), the first one 4: the large query component is about 15.7."""
    x = U.f64(W.hidden_bits(s, T, step=step))
    x[:, 0] = 4.0
    return _bits(x)


def _keys(s, seq, rise, spread, q=15.7):
    """Keys N(0, spread^2) whose scores carry an offset of rise[position] powers of two, for a large query component `q`."""
    rng = np.random.default_rng([s.seed, seq])
    k = rng.standard_normal((len(rise), s.Hkv, s.d)) * spread
    k[:, :, s.d // 2 - 1] = (np.asarray(rise) / (q / np.sqrt(s.d) * np.log2(np.e)))[:, None]
    k[:, :, s.d - 1] = 0.0
    return _bits(k)


def _run(torch, s, rows, caches, xbits):
    """One layer over sequences of `rows` new tokens each on the given caches ([(key bits, value bits)])."""
    n = len(caches)
    room = max(len(k) for k, _ in caches) + rows
    inst = U.make_instance(s, max_seqs=n, max_seq_len=room, max_tokens=n * rows, kv_tokens=n * (room + 32))
    inst.load_layer(0, inst.pinned_blob(inst.pack_layer(_layer(s))))
    for i, (k, v) in enumerate(caches):
        inst.kv_reserve(i, len(k) + rows)
        inst.kv_write(0, i, 0, len(k), k, v)
    x = U.to_device(xbits, False)
    torch.cuda.synchronize()
    inst.run_layers(0, 1, inst.batch([rows * i for i in range(n + 1)], list(range(n)), [len(k) for k, _ in caches]), x)
    inst.sync()
    got = U.from_device(x)
    inst.close()
    return got


def _oracle(s, rows, caches, xbits):
    okv = O.OracleKV()
    for i, (k, v) in enumerate(caches):
        okv.put(0, i, U.f64(k), U.f64(v))
    n = len(caches)
    return O.run_layers(U.oracle_shape(s), {0: U.oracle_weights(_layer(s))}, 0, 1, U.f64(xbits),
                        O.OracleBatch([rows * i for i in range(n + 1)], list(range(n)), [len(k) for k, _ in caches]), okv)


# rows per sequence and sequences: at most 64 rows in all (the projection comes as partial sums) and more, one key set and two
GRIDS = [(40, 1), (100, 1), (10, 6), (30, 6)]


@pytest.mark.parametrize("rows,seqs", GRIDS)
@pytest.mark.parametrize("d", [64, 128])
def test_rows_do_not_depend_on_the_rows_behind_them(torch, d, rows, seqs):
    """The same prompt's first rows come out the same bits whatever follows them in the batch of the same size.  Maxima rise
    by about 7 powers of two per 64 keys, by more or by less from row to row."""
    s = STEEP[d]
    keys = 704
    rise = 7.0 * (np.arange(keys) // 64)
    rng = np.random.default_rng(d)
    caches = [(_keys(s, i, rise, 0.5), _bits(rng.standard_normal((keys, s.Hkv, s.d)))) for i in range(seqs)]
    x = _hidden(s, rows * seqs, 1)
    y = _hidden(s, rows * seqs, 2)
    keep = rows // 2 - 4
    head = np.arange(rows * seqs) % rows < keep
    y[head] = x[head]
    assert np.array_equal(_run(torch, s, rows, caches, x)[head], _run(torch, s, rows, caches, y)[head])


@pytest.mark.parametrize("rows,seqs", GRIDS)
@pytest.mark.parametrize("d", [64, 128])
def test_large_values_stay_finite(torch, d, rows, seqs):
    """Weights relative to the row's own maximum sum up to the number of keys that count at most, here 2^12 - 64, so values
    of 2^112 stay within fp32, also where all keys but the first 64 score six powers of two above those."""
    s = STEEP[d]
    keys = 4096
    rise = np.where(np.arange(keys) < 64, 0.0, 6.0)
    caches = [(_keys(s, i, rise, 0.0), _bits(np.full((keys, s.Hkv, s.d), 2.0 ** 112))) for i in range(seqs)]
    x = _hidden(s, rows * seqs, 1)
    got = _run(torch, s, rows, caches, x)
    assert np.isfinite(got).all()
    assert U.rel_err(got, _oracle(s, rows, caches, x)) <= U.BF16_TOL


@pytest.mark.parametrize("d", [64, 128])
def test_decode_weights_below_the_normal_range_count(torch, d):
    """Single new tokens: weights 2^-129 of the largest one, which fp32 and bf16 hold as denormals, on values of 2^126, next to
    a largest one whose value is zero.  The offset comes from a query component of bf16, itself the product of a bf16
    value and a weight and then rotated: three roundings of 2^-9 on 129 powers of two, a factor of 2^0.76 at most."""
    s = STEEP[d]
    keys = 40
    rise = np.where(np.arange(keys) == 7, 65.0, -64.0)
    v = np.full((keys, s.Hkv, s.d), 2.0 ** 126)
    v[7] = 0.0
    x = _hidden(s, 3, 1)
    q = 4.0 * O.rmsnorm(U.f64(x), U.f64(_layer(s)["g1"]), s.eps)[:, 0]
    caches = [(_keys(s, i, rise, 0.0, q[i]), _bits(v)) for i in range(3)]
    got, want = _run(torch, s, 1, caches, x), _oracle(s, 1, caches, x)
    plain = _oracle(s, 1, [(k, _bits(np.zeros_like(v))) for k, _ in caches], x)
    large = np.abs(want - plain) > 0.5 * np.abs(want - plain).max()
    factor = (got - plain)[large] / (want - plain)[large]
    assert 2.0 ** -0.8 < factor.min() and factor.max() < 2.0 ** 0.8, (factor.min(), factor.max())


@pytest.mark.parametrize("d,prompt,single", [(64, 0, 60), (128, 0, 60), (64, 4, 60), (128, 40, 80), (64, 0, 130), (128, 0, 130)])
def test_many_decode_workgroups(torch, d, prompt, single):
    """Above 9600 workgroups per query head of a kv head the single new tokens are appended by a launch of its own.  The same batch in
    two halves takes the other kernel: same cache, bit for bit where the projection's plan is the same (up to 64 rows), and the
    same output within the gates; four sequences against the oracle.  60 sequences have more than four chunks each on average, 80
    and 130 fewer: their queries reach the products in different ways."""
    s = W.DecoderShape("wide%d" % d, L=1, H=512, Hq=40, Hkv=40, d=d, F=256, rope_base=10000.0, seed=90 + d)
    rng = np.random.default_rng([d, single])
    edges = [1023, 1024, 1055, 1056, 1279, 1280, 1281]
    before = (edges + rng.integers(1030, 1400, single - len(edges)).tolist()) if single <= 64 else \
             (edges + rng.integers(513, 800, single - len(edges)).tolist())
    news = [1] * single + ([prompt] if prompt else [])
    befores = before + ([700] if prompt else [])
    assert (sum(b // 256 + 1 for b in before) > 4 * single) == (single == 60)
    assert sum(b // 256 + 1 for b in before) * 40 > 9600 > sum(b // 256 + 1 for b in before[:(single + 1) // 2]) * 40
    n, T = len(news), sum(news)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    caches = [[torch.randn(b * s.Hkv * s.d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2)] for b in befores]
    start = np.concatenate([[0], np.cumsum(news)]).astype(int)
    xbits = W.hidden_bits(s, T, step=5, scale=1.0 / 16)
    bits = W.layer_weights_bits(s, 0)

    def run(parts):
        inst = U.make_instance(s, max_seqs=n, max_seq_len=max(befores) + 64, max_tokens=T, kv_tokens=sum(befores) + 96 * n)
        inst.load_layer(0, inst.pinned_blob(inst.pack_layer(bits)))
        for i, (k, v) in enumerate(caches):
            inst.kv_reserve(i, befores[i] + news[i])
            inst.kv_write(0, i, 0, befores[i], k, v)
        out = np.zeros((T, s.H))
        for ids in parts:
            q = np.concatenate([[0], np.cumsum([news[i] for i in ids])])
            rows = np.concatenate([np.arange(start[i], start[i + 1]) for i in ids])
            x = U.to_device(xbits[rows], False)
            torch.cuda.synchronize()
            inst.run_layers(0, 1, inst.batch(q, list(ids), [befores[i] for i in ids]), x)
            inst.sync()
            out[rows] = U.from_device(x)
        new = []
        for i in range(n):
            kv = [np.zeros((news[i], s.Hkv, s.d), dtype=np.uint16) for _ in range(2)]
            inst.kv_read(0, i, befores[i], news[i], *kv)
            new.append(kv)
        inst.close()
        return out, new

    half = (single + 1) // 2
    got, kv = run([range(n)])
    want, kv_want = run([range(half), range(half, n)])
    assert U.rel_err(got, want) <= U.BF16_TOL
    U.assert_rms(got, want, U.RMS_BF16)
    for a, b in zip(kv, kv_want):
        for x, y in zip(a, b):
            if T <= 64:
                assert np.array_equal(x, y)
            else:
                assert U.rel_err(U.f64(x), U.f64(y)) <= U.BF16_TOL
    okv, ids = O.OracleKV(), [1, 3, 5, n - 1]
    for j, i in enumerate(ids):
        k, v = (t.view(torch.int16).cpu().numpy().view(np.uint16).reshape(befores[i], s.Hkv, s.d) for t in caches[i])
        okv.put(0, j, U.f64(k), U.f64(v))
    rows = np.concatenate([np.arange(start[i], start[i + 1]) for i in ids])
    want = O.run_layers(U.oracle_shape(s), {0: U.oracle_weights(bits)}, 0, 1, U.f64(xbits[rows]),
                        O.OracleBatch(list(np.concatenate([[0], np.cumsum([news[i] for i in ids])])), [0, 1, 2, 3], [befores[i] for i in ids]), okv)
    assert U.rel_err(got[rows], want) <= U.BF16_TOL
    U.assert_rms(got[rows], want, U.RMS_BF16)
    for j, i in enumerate(ids):
        for g, o in zip(kv[i], okv.get(0, j, s.Hkv, s.d)):
            assert U.rel_err(U.f64(g), o[befores[i]:]) <= U.BF16_TOL


def _tile(keys):
    return np.arange(keys) // 64


# offsets of the keys, in powers of two, by KV tile of 64 positions
RISES = {
    "rising": lambda k: 12.0 * _tile(k),                                    # every tile moves every row's maximum
    "falling": lambda k: 12.0 * (_tile(k).max() - _tile(k)),
    "odd tiles": lambda k: np.where(_tile(k) % 2 == 1, 40.0, 0.0),          # two key sets: the second one's dominate
    "even tiles": lambda k: np.where(_tile(k) % 2 == 0, 40.0, 0.0),         # and vanish
    "last key": lambda k: np.where(np.arange(k) == k - 1, 60.0, 0.0),
    "rising by one": lambda k: 1.0 * _tile(k),                              # the sums of many tiles stay in the result
}


@pytest.mark.parametrize("rows,seqs", GRIDS)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rise", RISES, ids=lambda r: r.replace(" ", "_"))
def test_maxima_that_move_from_tile_to_tile(torch, rise, d, rows, seqs):
    """The sums of earlier keys are rescaled by far from one, by one and by nothing, and two key sets meet with references far
    apart.  Score differences up to 12 powers of two reach the result (2^-12 is below bf16's half ulp of the sum); they come
    from a query component of three bf16 roundings, 12 * 3 * 2^-9 = 0.07 powers of two or 5 % of a term of weight 2^-12, and the
    differences of a rising-by-one row from 11: below the gates everywhere."""
    s = STEEP[d]
    keys = 704
    rng = np.random.default_rng([d, rows])
    caches = [(_keys(s, i, RISES[rise](keys), 0.5), _bits(rng.standard_normal((keys, s.Hkv, s.d)))) for i in range(seqs)]
    x = _hidden(s, rows * seqs, 3)
    got, want = _run(torch, s, rows, caches, x), _oracle(s, rows, caches, x)
    assert U.rel_err(got, want) <= U.BF16_TOL
    U.assert_rms(got, want, U.RMS_BF16)
