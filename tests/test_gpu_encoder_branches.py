"""The encoders' branches against the oracle, blocks and meta words bit-exact: a workgroup per group and the bulk kernels
(one, two, four tiles of patterns; 32 groups of the full search and 16 of the min/max selector at a time, ragged ends),
groups for which the search's tables do not hold, patterns with crowded or equal centroids, codes beyond 8 bits."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2505_06901_amd as E  # noqa: E402
from test_paper_block_pins import _model as pb_model  # noqa: E402


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def model_tables(S, seed, long_codes=False):
    """Patterns of every width: spread over [-1, 1], crowded around 0, with equal neighbours, all equal."""
    from oracle import oracle as O
    rng = np.random.default_rng(seed)
    cent = np.sort(rng.uniform(-1, 1, (S, 16)) * 10.0 ** rng.uniform(-2.5, 0, (S, 1)), axis=1)
    cent[rng.random((S, 16)) < 0.1] = 0.25
    cent[S // 2, 5:9] = cent[S // 2, 5]
    if S > 2:
        cent[S - 1] = 0.5
    cent = np.sort(cent, axis=1).astype(np.float16)
    lens = np.zeros((S, 16), np.uint8)
    for p in range(S):
        counts = np.array([int((3.0 if long_codes else 1.5) ** k) + 1 for k in range(16)], np.uint64)[rng.permutation(16)]
        lens[p] = O.limited_lengths(counts, 12 if long_codes else 8)
    return cent, lens


def groups(cent, n, seed):
    """Values near a pattern's centroids and Gaussian ones, scales over the whole FP16 range, and degenerate groups."""
    rng = np.random.default_rng(seed)
    c = cent.astype(np.float64)[rng.integers(0, len(cent), n)]
    x = np.take_along_axis(c, rng.integers(0, 16, (n, 128)), axis=1)
    odd = rng.random(n) < 0.5
    x[odd] = rng.standard_normal((odd.sum(), 128)) / 3
    x = x * (1 + 0.01 * rng.standard_normal((n, 128))) * 10.0 ** rng.uniform(-6, 4, (n, 1))
    x = np.clip(x, -65504, 65504).astype(np.float16)
    edge = [np.zeros(128), -np.zeros(128), np.full(128, 6e-8), np.full(128, -65504.0), np.linspace(-1, 1, 128), np.linspace(-1, 1, 128) * 4.88e-4,
            np.linspace(-1, 1, 128) * 4.9e-4, np.where(np.arange(128) == 77, 1000.0, 3e-8), np.repeat([0.5, -0.5], 64)]
    for i, e in enumerate(edge):
        x[(i * 37) % n] = e.astype(np.float16)
    return x


@pytest.mark.parametrize("S,n,long_codes", [(1, 1, False), (3, 47, True), (16, 31, False), (16, 4001, False), (17, 2405, True), (33, 3000, False),
                                            (48, 33, False), (64, 1201, True), (64, 2113, False), (64, 20011, False),
                                            # a workgroup per group up to 7, 4, 3 and 2 of them for each of 256 compute units
                                            (8, 1792, True), (8, 1793, False), (20, 1024, False), (20, 1025, True), (40, 768, False), (40, 769, False), (64, 512, False),
                                            (64, 513, True)])
def test_encode_and_minmax(dev, S, n, long_codes):
    from oracle import oracle as O
    cent, lens = model_tables(S, S, long_codes)
    m = E.ecco_model_to_device(E.ecco_model_create(cent, lens), 0)
    x = groups(cent, n, n)
    t = torch.from_numpy(np.concatenate([np.zeros(2, np.float16), x.reshape(-1)])).to(dev)[2:].view(n, 128)  # 4-byte aligned only
    for name, want in (("full", O.encode(cent.view(np.uint16), lens, x.view(np.uint16))), ("minmax", O.encode_minmax(cent.view(np.uint16), lens, x.view(np.uint16)))):
        blocks, meta = (E.ecco_encode if name == "full" else E.ecco_encode_minmax)(m, t)
        assert np.array_equal(meta.cpu().numpy().view(np.uint32), want[1]), name
        assert np.array_equal(blocks.cpu().numpy(), want[0]), name


@pytest.mark.parametrize("B,H,Sk,Sv", [(3, 5, 16, 64), (7, 37, 33, 16), (16, 64, 64, 16), (16, 96, 3, 17), (8, 32, 64, 5), (9, 32, 64, 48)])
@pytest.mark.parametrize("minmax", [False, True])
def test_append_with_unlike_models(dev, B, H, Sk, Sv, minmax):
    """Keys and values under models of different sizes; sequences whose position lies outside the cache write nothing."""
    from oracle import oracle as O
    T = 3
    models, new, want = [], [], []
    for S, seed in ((Sk, 1), (Sv, 2)):
        cent, lens = model_tables(S, seed)
        models.append(E.ecco_model_to_device(E.ecco_model_create(cent, lens), 0))
        x = groups(cent, B * H, seed)
        new.append(torch.from_numpy(x.reshape(B, H, 128)).to(dev))
        want.append((O.encode_minmax if minmax else O.encode)(cent.view(np.uint16), lens, x.view(np.uint16)))
    at = np.arange(B, dtype=np.int32) % 5 - 1
    caches = [torch.full((B, H, T, 64), 0xA5, dtype=torch.uint8, device=dev), torch.full((B, H, T), -3, dtype=torch.int32, device=dev),
              torch.full((B, H, T, 64), 0xA5, dtype=torch.uint8, device=dev), torch.full((B, H, T), -3, dtype=torch.int32, device=dev)]
    (E.ecco_kv_append_minmax if minmax else E.ecco_kv_append)(*models, *new, *caches, torch.from_numpy(at).to(dev), B, H, T)
    for (ob, om), blocks, meta in zip(want, caches[::2], caches[1::2]):
        eb, em = np.full((B, H, T, 64), 0xA5, np.uint8), np.full((B, H, T), -3, np.int32)
        for b in range(B):
            if 0 <= at[b] < T:
                eb[b, :, at[b]] = ob.reshape(B, H, 64)[b]
                em[b, :, at[b]] = om.view(np.int32).reshape(B, H)[b]
        assert np.array_equal(blocks.cpu().numpy(), eb) and np.array_equal(meta.cpu().numpy(), em)


@pytest.mark.parametrize("S,n,texp", [(1, 1, -6), (16, 33, -9), (31, 1000, -8), (48, 65, -7), (64, 16421, -9)])
def test_self_contained_block(dev, S, n, texp):
    from oracle import paper_block as P
    om = pb_model(P, S=S, texp=texp, seed=S)
    m = E.ecco_pb_model_to_device(E.ecco_pb_model_create(om.cent, om.lens, om.kp_lens, om.texp), 0)
    x = groups(np.pad(om.cent.view(np.float16), ((0, 0), (0, 1)), mode="edge"), n, n)
    want = P.encode(om, x.view(np.uint16))
    assert np.array_equal(E.ecco_pb_encode(m, torch.from_numpy(x).to(dev)).cpu().numpy(), want)


def hard_groups(n, seed):
    """What the tables of the search do not serve, side by side in the wavefronts: all-zero groups (both signs), scales below
    2^-11 down to the smallest FP16 value, groups in which one value is far larger than the rest; ordinary ones between them."""
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((n, 128)) * 0.02
    kind = rng.integers(0, 8, n)
    x[kind == 0] = 0.0
    x[kind == 1] *= -0.0
    x[kind == 2] *= 2.0 ** -rng.uniform(5, 18, (n, 1))[kind == 2]
    k = np.flatnonzero((kind == 3) | (kind == 4))
    x[k, rng.integers(0, 128, k.size)] = 10.0 ** rng.uniform(-0.5, 2, k.size) * rng.choice([-1, 1], k.size)
    x[kind == 5] = np.sign(x[kind == 5]) * 6e-8
    return x.astype(np.float16)


def crowded_tables(S, seed):
    """Patterns of such groups: most centroids within a few hundredths of 0, some equal."""
    rng = np.random.default_rng(seed)
    cent = rng.standard_normal((S, 16)) * 10.0 ** rng.uniform(-3, -1, (S, 1))
    cent[:, 0], cent[:, 15] = -1, 1
    cent[rng.random((S, 16)) < 0.05] = 0.0
    return np.sort(np.clip(cent, -1, 1), axis=1).astype(np.float16)


@pytest.mark.parametrize("S,n", [(1, 3001), (2, 3002), (5, 2701), (16, 2001), (33, 1999), (63, 1031), (64, 4099)])
def test_value_by_value(dev, S, n):
    """Rows that leave the tables for the search over all centroids, alone in their wavefront and side by side; pattern
    counts that do not fill the search's last four."""
    from oracle import oracle as O
    from oracle import paper_block as P
    cent, x = crowded_tables(S, S), hard_groups(n, n)
    lens = np.full((S, 16), 4, np.uint8)
    m = E.ecco_model_to_device(E.ecco_model_create(cent, lens), 0)
    t = torch.from_numpy(x).to(dev)
    for encode, oracle_encode in ((E.ecco_encode, O.encode), (E.ecco_encode_minmax, O.encode_minmax)):
        want = oracle_encode(cent.view(np.uint16), lens, x.view(np.uint16))
        blocks, meta = encode(m, t)
        assert np.array_equal(meta.cpu().numpy().view(np.uint32), want[1])
        assert np.array_equal(blocks.cpu().numpy(), want[0])
    om = pb_model(P, S=S, texp=-9, seed=S)
    om.cent[:] = cent[:, :15].view(np.uint16)
    pm = E.ecco_pb_model_to_device(E.ecco_pb_model_create(om.cent, om.lens, om.kp_lens, om.texp), 0)
    assert np.array_equal(E.ecco_pb_encode(pm, t).cpu().numpy(), P.encode(om, x.view(np.uint16)))


@pytest.mark.parametrize("S,alike,n", [(17, 3, 1003), (33, 16, 2001), (64, 2, 1501), (64, 16, 2113), (64, 40, 999), (64, 64, 515)])
def test_patterns_dealt_out(dev, S, alike, n):
    """Patterns of which up to `alike` are the same, so that as many are left over from the bounds and tie, the lowest of them wins,
    beside groups with one left, none (all zero) and scales the tables do not serve: the patterns of a wavefront's four groups are
    rated by whichever row is free."""
    from oracle import oracle as O
    from oracle import paper_block as P
    rng = np.random.default_rng(S + alike)
    some = np.sort(rng.standard_normal((S, 16)) / 3, axis=1)
    some[:, 0], some[:, 15] = -1, 1
    some = np.sort(np.clip(some, -1, 1), axis=1).astype(np.float16)
    cent = some[np.minimum(np.arange(S), np.maximum(0, np.arange(S) - alike + 1))][rng.permutation(S)]  # the first one `alike` times
    lens = np.full((S, 16), 4, np.uint8)
    x = rng.standard_normal((n, 128)) * 0.02
    own = rng.random(n) < 0.5
    x[own] = some[0].astype(np.float64)[rng.integers(0, 16, (own.sum(), 128))] * 0.07 * (1 + 0.001 * rng.standard_normal((own.sum(), 128)))
    x[rng.random(n) < 0.1] = 0.0
    x[rng.random(n) < 0.1] *= 2.0 ** -9
    x = x.astype(np.float16)
    t = torch.from_numpy(x).to(dev)
    m = E.ecco_model_to_device(E.ecco_model_create(cent, lens), 0)
    want = O.encode(cent.view(np.uint16), lens, x.view(np.uint16))
    blocks, meta = E.ecco_encode(m, t)
    assert np.array_equal(meta.cpu().numpy().view(np.uint32), want[1])
    assert np.array_equal(blocks.cpu().numpy(), want[0])
    om = pb_model(P, S=S, texp=-9, seed=S)
    om.cent[:] = cent[:, :15].view(np.uint16)
    pm = E.ecco_pb_model_to_device(E.ecco_pb_model_create(om.cent, om.lens, om.kp_lens, om.texp), 0)
    assert np.array_equal(E.ecco_pb_encode(pm, t).cpu().numpy(), P.encode(om, x.view(np.uint16)))


def test_no_input_is_far_slower(dev):
    """Encoding must not collapse on padding (all-zero groups), on tiny scales or on groups that one value dominates: against
    ordinary weights at most 3 times for zeros (as fast, when measured) and 15 times where every value is compared with every
    centroid of all 64 patterns (6 to 9 times, when measured)."""
    from paper_2505_06901_amd import workloads as W
    n = 65536

    def outliers(rows, seed):
        x = np.random.default_rng(seed).standard_normal((rows, 128)) * 0.02
        x[:, 7] = 6.0
        return x.astype(np.float16)

    def time_of(call):
        call()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = float("inf")
        for _ in range(5):
            a.record(); call(); b.record(); b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    weights = W.weight_matrix(2048, 128, 0.02, 1e-3, 10.0, 1)
    w = torch.from_numpy(W.weight_matrix(n, 128, 0.02, 1e-3, 10.0, 2)).to(dev)
    tiny = (w.float() / w.float().abs().amax(1, keepdim=True) * 2.0**-20).half()
    blocks, meta = torch.empty((n, 64), dtype=torch.uint8, device=dev), torch.empty((n,), dtype=torch.int32, device=dev)
    out = torch.from_numpy(outliers(n, 4)).to(dev)
    m, mo = (E.ecco_model_to_device(E.ecco_fit_patterns(c, 64, 12, 1), 0) for c in (weights, outliers(2048, 3)))
    p, po = (E.ecco_pb_model_to_device(E.ecco_pb_fit(c, 64, 1), 0) for c in (weights, outliers(2048, 3)))
    for name, mm, mo, call in (("full", m, mo, lambda model, x: E.ecco_encode(model, x, blocks, meta)),
                               ("self-contained", p, po, lambda model, x: E.ecco_pb_encode(model, x, blocks))):
        usual = time_of(lambda: call(mm, w))
        assert time_of(lambda: call(mm, torch.zeros_like(w))) <= 3 * usual, name
        assert time_of(lambda: call(mm, tiny)) <= 15 * usual, name
        assert time_of(lambda: call(mo, out)) <= 15 * usual, name


@pytest.mark.parametrize("S", [1, 2, 5, 16, 63])
def test_minmax_bin_edges(dev, S):
    """Values on either side of every edge of the min/max selector's bins and of every midpoint between centroids, which lie
    far apart, a few per bin or many, at the smallest and largest scales of its table and across 2^15, where the factor
    onto its axis becomes a subnormal."""
    from oracle import oracle as O
    rng = np.random.default_rng(S)
    cent = crowded_tables(S, S + 100)
    cent[::3] = model_tables(S, S)[0][::3]
    lens = np.full((S, 16), 4, np.uint8)
    edges = (2.0 ** (np.arange(128) // 16 - 7) * (1 + np.arange(128) % 16 / 16) - 2.0 ** -7) / 1.988
    c = cent.astype(np.float64)
    marks = np.concatenate([edges, -edges, ((c[:, 1:] + c[:, :-1]) / 2).reshape(-1), c.reshape(-1)])
    n = 2048
    scale = np.array([2.0 ** -11, 2.0 ** -11 * 1.001, 0.02, 1.0, 3.3, 32752.0, 32800.0, 49152.0, 65504.0])[rng.integers(0, 9, n)].astype(np.float16)
    x = (rng.choice(marks, (n, 128)) * scale[:, None].astype(np.float64)).astype(np.float16)
    x = (x.view(np.int16) + np.where(x == 0, 0, rng.integers(-2, 3, x.shape)).astype(np.int16)).view(np.float16)  # up to two steps off
    x = np.where(np.abs(x) <= scale[:, None], x, scale[:, None])  # steps beyond 65504 are no numbers
    x[np.arange(n), rng.integers(0, 128, n)] = scale * rng.choice([-1, 1], n)
    m = E.ecco_model_to_device(E.ecco_model_create(cent, lens), 0)
    want = O.encode_minmax(cent.view(np.uint16), lens, x.view(np.uint16))
    blocks, meta = E.ecco_encode_minmax(m, torch.from_numpy(x).to(dev))
    assert np.array_equal(meta.cpu().numpy().view(np.uint32), want[1])
    assert np.array_equal(blocks.cpu().numpy(), want[0])


def offset_tables(S, seed):
    """Patterns of groups with a common offset: all centroids between half the scale and the scale, of one sign."""
    rng = np.random.default_rng(seed)
    cent = np.sort(rng.uniform(0.55, 1, (S, 16)), axis=1) * rng.choice([-1, 1], (S, 1))
    return np.sort(cent, axis=1).astype(np.float16)


def offset_groups(n, seed):
    rng = np.random.default_rng(seed)
    x = (1 + 0.1 * rng.standard_normal((n, 128))) * rng.choice([-1, 1], (n, 1)) * 10.0 ** rng.uniform(-5, 4, (n, 1))
    x[rng.random(n) < 0.1] *= 0.0
    return np.clip(x, -65504, 65504).astype(np.float16)


@pytest.mark.parametrize("S,n,long_codes", [(1, 2001, False), (3, 1999, True), (16, 4001, False), (63, 1601, False), (64, 2113, True)])
def test_minmax_uniform_bins(dev, S, n, long_codes):
    """Models whose centroids the min/max selector's bins crowd use the uniform ones: the edges of those and every midpoint
    between centroids, values around them, scales over the whole FP16 range; and an append under such a model beside one that does not."""
    from oracle import oracle as O
    rng = np.random.default_rng(S)
    cent, lens = offset_tables(S, S), model_tables(S, S, long_codes)[1]
    m = E.ecco_model_to_device(E.ecco_model_create(cent, lens), 0)
    c = cent.astype(np.float64)
    marks = np.concatenate([(256.0 * np.arange(257) - 32768) / 32700, ((c[:, 1:] + c[:, :-1]) / 2).reshape(-1), c.reshape(-1)])
    x = np.concatenate([offset_groups(n // 2, n), np.clip(rng.choice(marks, (n - n // 2, 128)), -1, 1) * 10.0 ** rng.uniform(-5, 4, (n - n // 2, 1))])
    x = np.clip(x, -65504, 65504).astype(np.float16)
    x[1::2, 0] = np.abs(x[1::2]).max(axis=1)
    want = O.encode_minmax(cent.view(np.uint16), lens, x.view(np.uint16))
    blocks, meta = E.ecco_encode_minmax(m, torch.from_numpy(x).to(dev))
    assert np.array_equal(meta.cpu().numpy().view(np.uint32), want[1])
    assert np.array_equal(blocks.cpu().numpy(), want[0])
    cent2, lens2 = model_tables(16, S + 1, long_codes)
    m2 = E.ecco_model_to_device(E.ecco_model_create(cent2, lens2), 0)
    B, H = 32, 40
    new = [x[:B * H], groups(cent2, B * H, S)]
    want = [O.encode_minmax(cent.view(np.uint16), lens, new[0].view(np.uint16)), O.encode_minmax(cent2.view(np.uint16), lens2, new[1].view(np.uint16))]
    caches = [torch.zeros((B, H, 1, 64), dtype=torch.uint8, device=dev), torch.zeros((B, H, 1), dtype=torch.int32, device=dev),
              torch.zeros((B, H, 1, 64), dtype=torch.uint8, device=dev), torch.zeros((B, H, 1), dtype=torch.int32, device=dev)]
    E.ecco_kv_append_minmax(m, m2, *(torch.from_numpy(a.reshape(B, H, 128)).to(dev) for a in new), *caches, torch.zeros(B, dtype=torch.int32, device=dev), B, H, 1)
    for (ob, om), blocks, meta in zip(want, caches[::2], caches[1::2]):
        assert np.array_equal(blocks.cpu().numpy().reshape(-1, 64), ob) and np.array_equal(meta.cpu().numpy().reshape(-1).view(np.uint32), om)


def test_minmax_with_a_common_offset(dev):
    """Groups with a common offset under a model fitted to such groups take at most 1.6 times as long as ordinary weights (1.1 to 1.2
    when measured; 2.4 where every wavefront compares its values with all centroids)."""
    from paper_2505_06901_amd import workloads as W
    n = 131072
    m = E.ecco_model_to_device(E.ecco_fit_patterns(W.weight_matrix(2048, 128, 0.02, 1e-3, 10.0, 1), 16, 12, 1), 0)
    w = torch.from_numpy(W.weight_matrix(n, 128, 0.02, 1e-3, 10.0, 2)).to(dev)
    mo = E.ecco_model_to_device(E.ecco_fit_patterns((1 + 0.1 * np.random.default_rng(1).standard_normal((2048, 128))).astype(np.float16), 16, 12, 1), 0)
    off = (1 + 0.1 * torch.randn(n, 128, device=dev, generator=torch.Generator(device=dev).manual_seed(2))).half()
    blocks, meta = torch.empty((n, 64), dtype=torch.uint8, device=dev), torch.empty((n,), dtype=torch.int32, device=dev)

    def time_of(model, x):
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                E.ecco_encode_minmax(model, x, blocks, meta)
            b.record(); b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    time_of(m, w)
    assert time_of(mo, off) <= 1.6 * time_of(m, w)
