"""GPU parity of the prefill-side token retention (Sec. 4.1; App. "Effect of Sentence Length") against the oracle:
skv_token_importance, skv_retain, skv_compact_pool, skv_build_semvec_layers, and the decode step on the retained pool.

Gates: importance within 2e-4 relative (+1e-7 of the largest value): both sides form the same exact bf16 products
(fp32 inputs: products exact to 2^-23) and differ in summation order and in exp2 vs exp; the retained set must equal
the oracle's rule applied to the GPU's own importance bit for bit, and may differ from the oracle's end-to-end set only
in tokens whose oracle importance is within 5e-4 relative of the cut ("documented tie"); offsets, lengths and compacted
rows bit-exact; decode on the retained pool to the usual attention tolerance.
"""
import math

import numpy as np
import pytest
import torch

from workload import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def U():
    import gpu_util
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return gpu_util


def _say(*a):
    print(*a, flush=True)


def _gpu_importance(U, ctx, q_obs, K, T, N):
    L = K.shape[0]
    alpha = torch.full((L, T - N), -5.0, dtype=torch.float32, device=U.DEV)
    nbytes = ctx.token_importance_work_bytes(T, N)
    assert nbytes > 0
    work = torch.empty(nbytes, dtype=torch.uint8, device=U.DEV)
    ctx.token_importance(q_obs, K, T, N, alpha, work)
    torch.cuda.synchronize()
    return alpha


IMP_CASES = [("bf16", 32, 8, 32, 1500), ("bf16", 8, 8, 32, 700), ("bf16", 16, 8, 32, 513), ("bf16", 64, 8, 32, 1100),
             ("bf16", 32, 8, 7, 530), ("bf16", 32, 8, 1, 300), ("f32", 32, 8, 16, 600), ("f32", 8, 2, 32, 257)]


@pytest.mark.parametrize("dtype,Hq,H,N,T", IMP_CASES, ids=[f"{c[0]}-Hq{c[1]}-H{c[2]}-N{c[3]}-T{c[4]}" for c in IMP_CASES])
def test_token_importance_matches_oracle(U, oracle32, dtype, Hq, H, N, T):
    _say("importance", dtype, Hq, H, N, T)
    L = 2
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype=dtype, len_dist=("uniform", 5, 30))
    lens = gen.sentence_lengths(wl.len_dist, T, seed=3)
    K = torch.stack([gen.kv_layer(lens, H, 128, wl.torch_dtype, 3, l)[0] for l in range(L)]).to(U.DEV)
    q_obs = gen.queries(L * Hq, N, 128, wl.torch_dtype, seed=4, device=U.DEV).view(L, Hq, N, 128)
    ctx = U.make_ctx(wl, T, len(lens), 16)
    alpha = _gpu_importance(U, ctx, q_obs, K, T, N).cpu().numpy()
    for l in range(L):
        ref = oracle32.token_importance(U.np_of(q_obs[l]), U.np_of(K[l]))
        err = np.abs(alpha[l] - ref)
        assert np.all(err <= 2e-4 * ref + 1e-7 * ref.max()), (l, float((err / (ref + 1e-30)).max()))
        assert np.all(alpha[l] >= 0)


@pytest.mark.parametrize("dtype,Hq,N,T", [("bf16", 32, 32, 2000), ("bf16", 64, 32, 1500), ("bf16", 32, 16, 1500), ("bf16", 8, 16, 1500),
                                          ("f32", 32, 32, 1100)])
def test_token_importance_with_logits_far_apart(U, oracle32, dtype, Hq, N, T):
    """Logits further apart than a float's exponent reaches, the first keys the smallest: sums relative to a row's first keys overflow."""
    _say("importance, logits far apart", dtype, Hq, N, T)
    wl = gen.CFG3.scaled(n_layers=1, n_q_heads=Hq, n_kv_heads=8, n_tokens=T, dtype=dtype, len_dist=("uniform", 5, 30))
    lens = gen.sentence_lengths(wl.len_dist, T, seed=3)
    K = gen.kv_layer(lens, 8, 128, wl.torch_dtype, 3, 0)[0][None].to(U.DEV) * 8
    K[:, :, :64] *= 0.01
    q_obs = gen.queries(Hq, N, 128, wl.torch_dtype, seed=4, device=U.DEV).view(1, Hq, N, 128) * 8
    alpha = _gpu_importance(U, U.make_ctx(wl, T, len(lens), 16), q_obs, K, T, N).cpu().numpy()
    ref = oracle32.token_importance(U.np_of(q_obs[0]), U.np_of(K[0]))
    # both sides sum 128 products in fp32 in partial sums up to 3500, each rounded by up to 2^-13: about 4e-4 in a logit (128 roundings of
    # random sign), over sqrt(D) 4e-5 of a probability, four times that at the worst of 10^6; measured 1e-4 (bf16), 1.8e-4 (fp32)
    assert np.all(np.abs(alpha[0] - ref) <= 4e-4 * ref + 1e-6 * ref.max())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Hq,N,T", [(8, 1, 2900), (8, 32, 2900), (16, 32, 2900), (32, 32, 2900), (64, 32, 2900),          # 1 row, then 32 to 256 rows per KV head
                                    (32, 32, 4500)])                                       # 128 rows in one sweep
def test_token_importance_precision_at_large_logits(U, dtype, Hq, N, T):
    """Logits that both sides form without rounding (two products of small whole numbers), 166 to 423 above zero in log2 units, within
    6 of each other: what is left is the softmax's own arithmetic, held against float64.  Bound, relative: the argument of exp2,
    at most 2^3, is rounded once (2^-22 * ln 2 = 1.7e-7), exp2 and 1 / sum to a unit each (1.8e-7), log2(e) / sqrt(D) is a
    float (2^-24 * 6 * ln 2 = 2.5e-7 over the spread), sums add a few 2^-24 (2e-7): below 1e-6."""
    H, D = 8, 128
    bases = [100, 100.5, 101, 111.5, 213, 255]                                              # a layer each
    L = len(bases)
    rng = np.random.default_rng(5)
    K = torch.zeros(L, H, T, D, dtype=torch.float32)
    v = rng.integers(0, 48, size=(L, H, T))
    K[..., 1] = torch.as_tensor(v, dtype=torch.float32)
    K[..., 0] = 13.0
    q = torch.zeros(L, Hq, N, D, dtype=torch.float32)
    q[..., 1] = 1.0
    for l, b in enumerate(bases):
        q[l, ..., 0] = b
    tt = torch.bfloat16 if dtype == "bf16" else torch.float32
    assert torch.equal(q.to(tt).float(), q) and torch.equal(K.to(tt).float(), K)
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype=dtype)
    _say("importance precision", dtype, Hq, N, T)
    got = _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q.to(tt).to(U.DEV), K.to(tt).to(U.DEV), T, N).cpu().numpy().astype(np.float64)
    worst = 0.0
    for l in range(L):
        want = np.zeros(T - N)
        for h in range(H):
            e = np.exp((v[l, h] - 47) / math.sqrt(D))                                       # the common part drops out
            z = np.cumsum(e)[T - N:]                                                        # window query n sees the keys 0 .. Tp + n
            want += (Hq // H) * e[:T - N] * (1.0 / z).sum()
        worst = max(worst, float(np.abs(got[l] / want - 1).max()))
    _say(f"  largest relative error {worst:.2e}")
    assert worst <= 1e-6


@pytest.mark.parametrize("dtype,Hq,N,per_cu", [("bf16", 32, 32, 3), ("bf16", 64, 16, 3), ("bf16", 64, 17, 2), ("bf16", 64, 32, 2), ("f32", 64, 32, 1)])
def test_token_importance_plans_for_the_blocks_that_fit(U, dtype, Hq, N, per_cu):
    """The scratch holds the plan: a partial per block of keys, whose length fills the chip's rounds of `per_cu` blocks (what LDS
    leaves room for: two of the 256-row form, three of the narrower ones, one for fp32) at the least rounds x (units of 128 keys + 2)."""
    L, H, T = 4, 8, 17000
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype=dtype)
    got = U.make_ctx(wl, T, 64, 16).token_importance_work_bytes(T, N)
    resident = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    units = -(-T // 128)
    chunks = lambda per: -(-units // per)
    per = min(range(1, min(256, units) + 1), key=lambda p: -(-L * H * chunks(p) // resident) * (p + 2))
    rows = next(r for r in (32, 64, 128, 256) if Hq // H * N <= r)
    want = 4 * (L * H * chunks(per) * rows * 2 + L * H * rows * 2 + L * H * (T - N))
    assert got == -(-want // 256) * 256

SWEEP_CASES = [(8, 32, 1023), (8, 32, 1025), (8, 1, 2), (8, 7, 40), (16, 32, 512), (16, 25, 513), (16, 32, 1057), (32, 32, 4096),
               (32, 24, 4353), (32, 32, 16384), (32, 32, 40), (32, 32, 255), (32, 32, 256), (32, 32, 257), (32, 17, 300), (32, 32, 1025)]


def _importance_inputs(U, L, Hq, H, N, T, seed=11):
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype="bf16")
    g = torch.Generator(device=U.DEV)
    g.manual_seed(seed)
    K = torch.empty(L, H, T, 128, dtype=torch.bfloat16, device=U.DEV).normal_(generator=g)
    q = torch.empty(L, Hq, N, 128, dtype=torch.bfloat16, device=U.DEV).normal_(generator=g)
    return wl, q, K


@pytest.mark.parametrize("limit", [None, 0])
@pytest.mark.parametrize("Hq,N,T", SWEEP_CASES, ids=[f"rows{c[0] // 8 * c[1]}-N{c[1]}-T{c[2]}" for c in SWEEP_CASES])
def test_token_importance_in_one_sweep(U, Hq, N, T, limit):
    """The one-sweep form at the edges of its chunks (1024, 512 or 256 keys), from one chunk to several rounds of them, against the two passes.
    Both form the same logits bit for bit; arguments of exp2 (up to 2^4 here) are rounded once to 2^-21 on each side, sums of T terms differ in
    order: 2^-20 * ln 2 + a few 2^-24 of a value, below 2e-6.  With a wait limit of zero every block leaves the work to the passes behind
    the sweep, which give their very bits; without one the sweep's own result arrives, which among so many values has other bits somewhere."""
    L, H = 36, 8                                                                            # 288 (layer, head) pairs
    _say("importance in one sweep", Hq, N, T, limit)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want = _gpu_importance(U, two, q, K, T, N)
    ctx = U.make_ctx(wl, T, 64, 16)
    if limit is not None:
        ctx.set_wait_limit(limit)
    for _ in range(3):                                                                      # launch numbers move on
        got = _gpu_importance(U, ctx, q, K, T, N)
        if limit == 0 and T > 8192 // Hq:                                                   # (a head in one chunk waits for nobody)
            assert torch.equal(got, want)
        if limit is None and T > 250:
            assert not torch.equal(got, want)
        rel = ((got - want).abs() / want.abs().clamp_min(1e-30)).max().item()
        assert rel <= 2e-6, rel
    if limit == 0:
        ctx.set_wait_limit(200000)
        rel = ((_gpu_importance(U, ctx, q, K, T, N) - want).abs() / want.abs().clamp_min(1e-30)).max().item()
        assert rel <= 2e-6, rel


@pytest.mark.parametrize("Hq,N,T", [(8, 32, 9000), (16, 32, 4300), (32, 32, 16384)])
@pytest.mark.parametrize("limit", [1, 3])
def test_token_importance_sweep_gives_up_on_the_way(U, Hq, N, T, limit):
    """So few polls that some blocks give up at one chunk, some at another, and some not at all: the launch ends, its numbers move on, and the result is
    that of the sweep or of the two passes behind it, call after call; without the limit the sweep runs again."""
    L, H = 36, 8
    _say("importance in one sweep, gives up on the way", Hq, N, T, limit)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want = _gpu_importance(U, two, q, K, T, N)
    ctx = U.make_ctx(wl, T, 64, 16)
    for polls in (limit, limit, limit, 200000):
        ctx.set_wait_limit(polls)
        assert ((_gpu_importance(U, ctx, q, K, T, N) - want).abs() / want.abs().clamp_min(1e-30)).max().item() <= 2e-6


@pytest.mark.parametrize("Hq", [8, 16, 32])                                                # chunks of 1024, 512 and 256 keys
def test_token_importance_sweep_with_infinities_and_nan(U, Hq):
    """A NaN or infinite logit, and keys that every row weighs zero: the places of NaN and the values are those of the two passes, to the bound above; that not all
    bits are shows whose result it is, layer by layer."""
    L, H, N, T = 4, 8, 32, 5000
    _say("importance in one sweep, special values", Hq)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    K[0, 1, 700] = float("nan")
    K[1, 2, 800, 3] = float("inf")
    K[2, :, 900:1900] = -200.0 * q[2, ::Hq // H, 0].float().sign().to(torch.bfloat16)[:, None]
    q[2] = q[2, ::Hq // H, :1].repeat_interleave(Hq // H, 0)                                # (every row of a head is the first)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want, got = _gpu_importance(U, two, q, K, T, N), _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q, K, T, N)
    assert torch.equal(want.isnan(), got.isnan())
    assert want[0].isnan().sum() == want[1].isnan().sum() == 1 and not want[2:].isnan().any()
    assert torch.all(want[2, 900:1900] == 0)
    for l in range(L):
        ok = ~want[l].isnan()
        assert torch.all((got - want)[l].abs()[ok] <= 2e-6 * want[l][ok] + 1e-30)
        assert not torch.equal(got[l][ok], want[l][ok]), l


@pytest.mark.parametrize("Hq", [8, 16, 32])
def test_token_importance_sweep_beyond_its_exponents(U, Hq):
    """Logits beyond what the words of the exchange hold, in one layer: the sweep gives up and the two passes do all layers, bit for bit."""
    L, H, N, T = 4, 8, 32, 5000
    _say("importance in one sweep, beyond its exponents", Hq)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    q[3, 5] *= 2.0 ** 15                                                                    # logits of some 10^5 in log2 units, words up to 65279
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want, got = _gpu_importance(U, two, q, K, T, N), _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q, K, T, N)
    assert torch.equal(got, want) and not want.isnan().any()


# a wave combines 16, 64 or 128 chunks in one round of loads and more in several: 16, 17, 64, 65 and 128 chunks of 256 keys, 137 of 512, 17 of 1024
@pytest.mark.parametrize("L,Hq,H,N,T", [(6, 4, 1, 32, 4096), (6, 4, 1, 32, 4097), (2, 4, 1, 32, 16384), (2, 4, 1, 32, 16400), (1, 4, 1, 32, 32768),
                                        (1, 2, 1, 32, 70001), (6, 1, 1, 32, 16500)])
def test_token_importance_sweep_combines_any_number_of_chunks(U, L, Hq, H, N, T):
    """Against the two passes, to the bound of test_token_importance_in_one_sweep; other bits show whose result it is."""
    _say("importance in one sweep, chunks", L, Hq, N, T)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want, got = _gpu_importance(U, two, q, K, T, N), _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q, K, T, N)
    assert ((got - want).abs() / want).max().item() <= 2e-6
    assert not torch.equal(got, want)


# 128 rows, 256 keys a chunk: 57 chunks a head fill 456 of the 512 blocks, 73 and 74 fill 511 and 444, 102 and 103 fill 510 and 412, 129 are too many
@pytest.mark.parametrize("L,chunks,sweeps", [(9, 57, True), (9, 73, True), (9, 74, False), (8, 74, True), (8, 102, True), (8, 103, False), (1, 128, True), (1, 129, False)])
def test_token_importance_sweep_where_whole_heads_fill_the_chip(U, L, chunks, sweeps):
    """Which of the two forms a launch takes, by its bits; the sweep to the bound of test_token_importance_in_one_sweep."""
    Hq, H, N, T = 32, 8, 32, 256 * chunks
    _say("importance in one sweep, whole heads", L, chunks)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want, got = _gpu_importance(U, two, q, K, T, N), _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q, K, T, N)
    assert torch.equal(got, want) == (not sweeps)
    assert ((got - want).abs() / want).max().item() <= 2e-6


@pytest.mark.parametrize("Hq", [8, 16, 32])                                                # chunks of 1024, 512 and 256 keys
@pytest.mark.parametrize("rise", [16, 40, 120, 250])
def test_token_importance_sweep_of_logits_that_rise(U, Hq, rise):
    """The first keys of some chunks, the first and the last among them, lie `rise` (log2 units) below the rest: sums relative to a chunk's first keys stay
    below 2^24 or pass it, or overflow.  Arguments of exp2 below 2^6 (below 2^8: results under 1e-19 of the others, held to 1e-30 in all) are rounded
    to 2^-19 on each side: 2 * 2^-19 * ln 2 = 2.6e-6 of a value, with sums in another order below 4e-6."""
    L, H, N, T = 4, 8, 32, 4120
    _say("importance in one sweep, rising logits", Hq, rise)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    q[..., 0] = 8.0
    K[..., 0] = 0.0
    low = -rise / (8 * 1.4426950408889634 / math.sqrt(128))
    for first in (0, 1024, 2304, 3072, 4096):
        K[:, ::2, first:first + 20, 0] = low
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want, got = _gpu_importance(U, two, q, K, T, N), _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q, K, T, N)
    assert torch.isfinite(got).all()
    assert torch.all((got - want).abs() <= 4e-6 * want + 1e-30)
    for l in range(L):
        assert not torch.equal(got[l], want[l])


@pytest.mark.parametrize("Hq", [8, 16, 32])                                                # a wave takes tiles of 16 keys, 64, 32 and 16 keys apart
@pytest.mark.parametrize("step", [20, 25, 30, 100])
def test_token_importance_sweep_of_logits_that_rise_tile_by_tile(U, Hq, step):
    """Every tile of a wave lies `step` (log2 units) above the one before it, so that references move up never, now and then or each time; in one layer all rows,
    in one a single row; in the others the steps begin late in the chunk, or are taken in the window's own.  The bound of
    test_token_importance_sweep_of_logits_that_rise."""
    L, H, N, T = 4, 8, 32, 4120
    _say("importance in one sweep, rising tiles", Hq, step)
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    apart = 512 // Hq
    tile = torch.arange(T, device=U.DEV) // apart % 16
    q[..., 0] = 0.0
    q[0, ..., 0] = 8.0
    q[1, ::Hq // H, 5, 0] = 8.0
    q[2:, ..., 0] = 8.0
    K[..., 0] = 0.0
    unit = step / (8 * 1.4426950408889634 / math.sqrt(128))
    K[0, ..., 0] = K[1, ..., 0] = (tile * unit).to(torch.bfloat16)
    K[2, ..., 0] = ((tile - 12).clamp_min(0) * unit).to(torch.bfloat16)
    K[3, :, T - 100:, 0] = (tile[T - 100:] * unit).to(torch.bfloat16)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want, got = _gpu_importance(U, two, q, K, T, N), _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q, K, T, N)
    assert torch.isfinite(got).all()
    for l in range(L):
        assert torch.all((got - want)[l].abs() <= 4e-6 * want[l] + 1e-30), l
        assert not torch.equal(got[l], want[l])


@pytest.mark.parametrize("Hq,keys", [(8, 64), (16, 32)])                                     # keys of a block's four or two waves, 16 each
def test_token_importance_sweep_of_a_wave_far_below_the_others(U, Hq, keys):
    """The 16 keys in `keys` that one wave of a block takes lie 2^31 and more (log2 units) below those of its other waves: they weigh nothing, the others what they weigh
    without them (logits within 6 of zero: the bound of test_token_importance_precision_at_large_logits)."""
    L, H, N, T, D = 4, 8, 32, 4128, 128
    _say("importance in one sweep, a wave far below", Hq)
    v = np.random.default_rng(Hq).integers(0, 48, size=(L, H, T))
    K = torch.zeros(L, H, T, D)
    K[..., 1] = torch.as_tensor(v, dtype=torch.float32)
    far = np.zeros(T, dtype=bool)
    far[1024:3072] = np.arange(1024, 3072) // 16 % (keys // 16) == 1
    K[:, :, far, 0] = -2.0 ** 24
    q = torch.zeros(L, Hq, N, D)
    q[..., 1] = 1.0
    q[..., 0] = 2.0 ** 20
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype="bf16")
    got = _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q.to(torch.bfloat16).to(U.DEV), K.to(torch.bfloat16).to(U.DEV), T, N).cpu().numpy().astype(np.float64)
    e = np.where(far, 0.0, np.exp((v - 47) / math.sqrt(D)))
    z = np.cumsum(e, axis=-1)[..., T - N:]
    want = (Hq // H * e[..., :T - N] * (1.0 / z).sum(-1, keepdims=True)).sum(1)
    assert np.all(got[:, far[:T - N]] == 0)
    assert np.all(np.abs(got - want) <= 1e-6 * want)


@pytest.mark.parametrize("Hq,keys", [(8, 64), (16, 32)])
def test_token_importance_sweep_of_a_wave_far_below_in_rounded_logits(U, Hq, keys):
    """As above, with logits that a float does not hold: rounded at 2^41 they differ by thousands of log2 units from the largest of their tile, rounded otherwise,
    and are nothing next to the others all the same."""
    L, H, N, T, D = 4, 8, 32, 4128, 128
    _say("importance in one sweep, a wave far below, rounded", Hq)
    rng = np.random.default_rng(Hq)
    v = rng.integers(0, 48, size=(L, H, T))
    K = torch.zeros(L, H, T, D)
    K[..., 1] = torch.as_tensor(v, dtype=torch.float32)
    far = np.zeros(T, dtype=bool)
    far[1024:3072] = np.arange(1024, 3072) // 16 % (keys // 16) == 1
    far[3088:3104] = True                                                                   # the first tile of a wave whose others are not far
    K[:, :, far, 0] = torch.as_tensor(-2.0 ** 17 * rng.integers(128, 256, size=(L, H, int(far.sum()))), dtype=torch.float32)
    q = torch.zeros(L, Hq, N, D)
    q[..., 1] = 1.0
    q[..., 0] = 2.0 ** 20
    assert torch.equal(K.to(torch.bfloat16).float(), K)
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype="bf16")
    got = _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q.to(torch.bfloat16).to(U.DEV), K.to(torch.bfloat16).to(U.DEV), T, N).cpu().numpy().astype(np.float64)
    e = np.where(far, 0.0, np.exp((v - 47) / math.sqrt(D)))
    z = np.cumsum(e, axis=-1)[..., T - N:]
    want = (Hq // H * e[..., :T - N] * (1.0 / z).sum(-1, keepdims=True)).sum(1)
    assert np.all(got[:, far[:T - N]] == 0)
    assert np.all(np.abs(got - want) <= 1e-6 * want)


# the last chunk holds 1, 16, 17, 40 or 60 keys (of 1024, 512 and 256), or is the only one
BELOW_ZERO = [(8, t) for t in (40, 1025, 1040, 1041, 1064, 1084, 4136)] + [(16, t) for t in (40, 513, 528, 529, 552, 572)] + [(32, t) for t in (40, 257, 272, 273, 296)]


@pytest.mark.parametrize("Hq,T", BELOW_ZERO, ids=[f"rows{4 * hq}-T{t}" for hq, t in BELOW_ZERO])
def test_token_importance_sweep_of_logits_far_from_zero(U, Hq, T):
    """A shift of a row's logits leaves its softmax alone, also where parts of a block see none of the last chunk's keys: all logits up to 423 below or
    above zero in log2 units, a layer each, products and sums exact as in test_token_importance_precision_at_large_logits, the window's own keys up to 2^6 times as
    heavy as the rest.  The bound of that test, for arguments of exp2 of up to 2^4 (rounded to 2^-21: 3.3e-7) and twice its spread (5e-7): 1.4e-6."""
    H, N, D = 8, 32, 128
    bases = [-255, -213, -181, -111.5, -101, -100.5, -90.5, -50, 0, 100.5, 181, 255]
    L = len(bases)                                                                          # 96 (layer, head) pairs: one chunk each is enough
    _say("importance in one sweep, logits far from zero", Hq, T)
    v = np.random.default_rng(T).integers(0, 48, size=(L, H, T))
    v[:, :, T - N:] += 48
    K = torch.zeros(L, H, T, D)
    K[..., 1] = torch.as_tensor(v, dtype=torch.float32)
    K[..., 0] = 13.0
    q = torch.zeros(L, Hq, N, D)
    q[..., 1] = 1.0
    q[..., 0] = torch.tensor(bases)[:, None, None]
    K16, q16 = K.to(torch.bfloat16), q.to(torch.bfloat16)
    assert torch.equal(K16.float(), K) and torch.equal(q16.float(), q)
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype="bf16")
    got = _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q16.to(U.DEV), K16.to(U.DEV), T, N).cpu().numpy().astype(np.float64)
    e = np.exp((v - 95) / math.sqrt(D))                                                     # the common part drops out
    z = np.cumsum(e, axis=-1)[..., T - N:]                                                  # window query n sees the keys 0 .. Tp + n
    want = (Hq // H * e[..., :T - N] * (1.0 / z).sum(-1, keepdims=True)).sum(1)
    worst = np.abs(got / want - 1).max(1)
    _say("  largest relative error of each layer", *(f"{x:.1e}" for x in worst))
    assert np.all(worst <= 1.4e-6)


@pytest.mark.parametrize("Hq", [8, 16, 32])                                                # chunks of 1024, 512 and 256 keys
@pytest.mark.parametrize("base", [-255, -100, 0, 100])
def test_token_importance_sweep_of_chunks_that_begin_with_infinite_keys(U, Hq, base):
    """Sixteen keys and more whose logits are -infinity, where a block, one of its waves or the window begins: they weigh nothing, and the keys behind them, up to 430
    from zero in log2 units, what they weigh without them.  The bound of test_token_importance_sweep_of_logits_far_from_zero."""
    L, H, N, T, D = 4, 8, 32, 4128, 128
    _say("importance in one sweep, infinite keys first", Hq, base)
    v = np.random.default_rng(Hq).integers(0, 48, size=(L, H, T))
    K = torch.zeros(L, H, T, D)
    K[..., 1] = torch.as_tensor(v, dtype=torch.float32)
    K[..., 0] = 13.0
    gone = np.zeros(T, dtype=bool)
    for first, last in ((0, 16), (1040, 1056), (2096, 2112), (3072, 3136), (4096, 4112)):
        gone[first:last] = True
    K[:, :, gone, 2] = -math.inf
    q = torch.zeros(L, Hq, N, D)
    q[..., 1:3] = 1.0
    q[..., 0] = base
    wl = gen.CFG3.scaled(n_layers=L, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype="bf16")
    got = _gpu_importance(U, U.make_ctx(wl, T, 64, 16), q.to(torch.bfloat16).to(U.DEV), K.to(torch.bfloat16).to(U.DEV), T, N).cpu().numpy().astype(np.float64)
    e = np.where(gone, 0.0, np.exp((v - 47) / math.sqrt(D)))
    z = np.cumsum(e, axis=-1)[..., T - N:]
    want = (Hq // H * e[..., :T - N] * (1.0 / z).sum(-1, keepdims=True)).sum(1)
    assert np.all(got[:, gone[:T - N]] == 0)
    assert np.all(np.abs(got - want) <= 1.4e-6 * want)


def test_token_importance_sweep_after_one_beyond_its_exponents(U):
    """A sweep that gave up over logits beyond the exponents of its words leaves words that no later launch takes for its own: here the place of the exponent
    alone would turn the tags of a first launch, 1 to 256, into those of the second."""
    L, Hq, H, N, T = 32, 8, 8, 32, 4128
    _say("importance in one sweep, after one beyond its exponents")
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want = _gpu_importance(U, two, q, K, T, N)
    ctx = U.make_ctx(wl, T, 64, 16)
    q_far, K_far = torch.zeros_like(q), torch.zeros_like(K)
    q_far[..., 0], K_far[..., 0] = 16384, 16064                                             # 2^25 and some thousands in log2 units
    _gpu_importance(U, ctx, q_far, K_far, T, N)
    got = _gpu_importance(U, ctx, q, K, T, N)
    assert ((got - want).abs() / want).max().item() <= 2e-6


def test_token_importance_sweeps_on_two_streams(U):
    """Two contexts whose sweeps meet on the GPU: each finds part of the compute units taken, its blocks wait or leave the work to the two passes;
    the results are those of a sweep alone to the bound of the test above."""
    L, Hq, H, N, T = 16, 8, 8, 32, 32768
    _say("importance in one sweep, two streams")
    work = []
    for seed in (1, 2):
        wl, q, K = _importance_inputs(U, L, Hq, H, N, T, seed=seed)
        ctx = U.make_ctx(wl, T, 64, 16)
        want = _gpu_importance(U, ctx, q, K, T, N)
        stream = torch.cuda.Stream()
        ctx.set_stream(stream.cuda_stream)
        scratch = torch.empty(ctx.token_importance_work_bytes(T, N), dtype=torch.uint8, device=U.DEV)
        work.append((ctx, q, K, torch.zeros_like(want), scratch, want, stream))
    torch.cuda.synchronize()
    for _ in range(5):
        for ctx, q, K, alpha, scratch, _, _ in work:
            ctx.token_importance(q, K, T, N, alpha, scratch)
    torch.cuda.synchronize()
    for _, _, _, alpha, _, want, _ in work:
        assert ((alpha - want).abs() / want).max().item() <= 2e-6


def test_importance_and_long_retention_in_a_graph(U):
    """The sweep and the retention of a long prompt recorded into a HIP graph: launch numbers, tags and counters live on the device, so that replays with
    calls of the same context in between give what direct calls give."""
    L, Hq, H, N, T, k = 4, 16, 8, 32, 30000, 3000
    _say("importance and retention in a graph")
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    seg = torch.arange(T, device=U.DEV, dtype=torch.int32) // 20
    S = int(seg[-1]) + 1
    ctx = U.make_ctx(wl, T, S, 16)
    work = torch.empty(ctx.token_importance_work_bytes(T, N), dtype=torch.uint8, device=U.DEV)

    def outputs():
        return (torch.zeros(L, T - N, device=U.DEV), torch.zeros(L, k, dtype=torch.int32, device=U.DEV), torch.zeros(L, dtype=torch.int32, device=U.DEV),
                torch.zeros(L, S + 1, dtype=torch.int32, device=U.DEV), torch.zeros(L, S, dtype=torch.int32, device=U.DEV))

    def call(alpha, keep, n_keep, off, ln):
        ctx.token_importance(q, K, T, N, alpha, work)
        ctx.retain(alpha, T - N, k, seg, S, keep, n_keep, off, ln)

    want, got = outputs(), outputs()
    call(*want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.set_stream(torch.cuda.current_stream().cuda_stream)
        call(*got)
    ctx.set_stream(torch.cuda.current_stream().cuda_stream)
    for _ in range(4):
        for t in got:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        eager = outputs()
        call(*eager)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(eager, want))


def test_token_importance_sweep_tags_start_again(U):
    """2^24 tags, one per (layer, head) and launch: with 2^19 pairs they are used up at the 32nd launch."""
    L, Hq, H, N, T = 8192, 64, 64, 2, 20
    _say("importance in one sweep, tags used up")
    wl, q, K = _importance_inputs(U, L, Hq, H, N, T)
    two = U.make_ctx(wl, T, 64, 16)
    two.set_single_launch(False)
    want = _gpu_importance(U, two, q, K, T, N)
    ctx = U.make_ctx(wl, T, 64, 16)
    first = _gpu_importance(U, ctx, q, K, T, N)
    assert ((first - want).abs() / want).max().item() <= 2e-6
    for _ in range(40):
        assert torch.equal(_gpu_importance(U, ctx, q, K, T, N), first)


FULL_IMP_CASES = [("bf16", 32, 8, 32, 32768), ("f32", 32, 8, 32, 32768), ("bf16", 8, 2, 32, 40100), ("f32", 4, 1, 32, 70001)]


@pytest.mark.parametrize("dtype,Hq,H,N,T", FULL_IMP_CASES, ids=[f"{c[0]}-Hq{c[1]}-H{c[2]}-N{c[3]}-T{c[4]}" for c in FULL_IMP_CASES])
def test_token_importance_and_retention_at_benchmark_size(U, oracle32, dtype, Hq, H, N, T):
    """The size the retention benchmark times (32768 tokens, 32/8 heads, a 32-token window) and longer prompts of few heads, whose rows are
    combined from up to 314 blocks of keys; most stages lie wholly before the window (no masking): one layer against the oracle, then
    the k = 4096 best tokens by the oracle's rule on the GPU's own importance, bit for bit."""
    _say("importance at size", dtype, Hq, H, N, T)
    wl = gen.CFG3.scaled(n_layers=1, n_q_heads=Hq, n_kv_heads=H, n_tokens=T, dtype=dtype)
    lens = gen.sentence_lengths(wl.len_dist, T, seed=5)
    K = gen.kv_layer(lens, H, 128, wl.torch_dtype, 5, 0)[0][None].to(U.DEV)
    q_obs = gen.queries(Hq, N, 128, wl.torch_dtype, seed=6, device=U.DEV).view(1, Hq, N, 128)
    S = len(lens)
    ctx = U.make_ctx(wl, T, S, 16)
    alpha_dev = _gpu_importance(U, ctx, q_obs, K, T, N)
    alpha = alpha_dev.cpu().numpy()
    ref = oracle32.token_importance(U.np_of(q_obs[0]), U.np_of(K[0]))
    err = np.abs(alpha[0] - ref)
    assert np.all(err <= 2e-4 * ref + 1e-7 * ref.max()), float((err / (ref + 1e-30)).max())
    assert np.all(alpha[0] >= 0)
    k, Tp = 4096, T - N
    seg = np.repeat(np.arange(S), lens).astype(np.int32)[:T]
    keep, n_keep, off, ln = _gpu_retain(U, ctx, alpha_dev, k, seg, S)
    want_keep, want_off, want_len = oracle32.retain(alpha[0], k, seg, S)
    assert n_keep[0] == len(want_keep) == min(k, Tp)
    assert np.array_equal(keep[0, :n_keep[0]], want_keep)
    assert np.array_equal(off[0], want_off) and np.array_equal(ln[0], want_len)
    # end to end against the oracle's own importance: the two sets may differ only in tokens at the cut
    ref_keep, _, _ = oracle32.retain(ref, k, seg, S)
    diff = np.setxor1d(want_keep, ref_keep)
    if len(diff):
        cut = np.sort(ref)[::-1][k - 1]
        _say(f"  retained sets differ in {len(diff)} tokens at the cut")
        assert np.all(np.abs(ref[diff] - cut) <= 5e-4 * cut), float(np.abs(ref[diff] - cut).max() / cut)


def _gpu_retain(U, ctx, alpha_dev, k, seg_id, S):
    L, Tp = alpha_dev.shape
    keep = U.empty_i32(L, max(k, 1), fill=-9)
    n_keep = U.empty_i32(max(L, 4), fill=-9)
    off = U.empty_i32(L, S + 1, fill=-9)
    ln = U.empty_i32(L, S, fill=-9)
    ctx.retain(alpha_dev, Tp, k, U.i32(seg_id), S, keep, n_keep, off, ln)
    torch.cuda.synchronize()
    return keep.cpu().numpy(), n_keep.cpu().numpy()[:L], off.cpu().numpy(), ln.cpu().numpy()


@pytest.mark.parametrize("Tp", [1, 2, 63, 1023, 1024, 1025, 5000, 40001])
def test_retain_bit_exact(U, oracle32, Tp):
    _say("retain Tp", Tp)
    L = 3
    rng = np.random.default_rng(Tp)
    alpha = rng.random((L, Tp)).astype(np.float32)
    alpha[1] = rng.choice(np.array([0.0, 0.125, 0.5, 2.0], np.float32), size=Tp)        # many exact ties
    alpha[2, rng.integers(0, Tp, max(Tp // 50, 1))] = np.nan
    alpha[2, rng.integers(0, Tp, max(Tp // 50, 1))] = -0.0
    lens = gen.sentence_lengths(("uniform", 1, 40), Tp + 8, seed=Tp)
    seg = np.repeat(np.arange(len(lens)), lens).astype(np.int32)
    S = len(lens)
    wl = gen.CFG3.scaled(n_layers=L)
    ctx = U.make_ctx(wl, Tp + 8, S, 16)
    a_dev = torch.from_numpy(alpha).to(U.DEV)
    for k in sorted({0, 1, Tp // 7, Tp // 2, Tp - 1, Tp, Tp + 3}):
        if k < 0:
            continue
        keep, n_keep, off, ln = _gpu_retain(U, ctx, a_dev, k, seg, S)
        for l in range(L):
            want_keep, want_off, want_len = oracle32.retain(alpha[l], k, seg, S)
            assert n_keep[l] == len(want_keep) == min(k, Tp)
            assert np.array_equal(keep[l, :n_keep[l]], want_keep), (k, l)
            assert np.all(keep[l, n_keep[l]:] == -9)                                       # nothing written past n_keep
            assert np.array_equal(off[l], want_off) and np.array_equal(ln[l], want_len), (k, l)


@pytest.mark.parametrize("Tp", [32768, 32769, 36001])
def test_retain_long_prompts_of_many_layers(U, oracle32, Tp):
    """More layers than the form of several blocks has scratch for: one block per layer, which holds 32768 tokens in registers and reads longer
    prompts again in every sweep."""
    _say("retain, 257 layers", Tp)
    L = 257
    rng = np.random.default_rng(Tp)
    lens = gen.sentence_lengths(("uniform", 1, 40), Tp + 8, seed=Tp)
    seg = np.repeat(np.arange(len(lens)), lens).astype(np.int32)
    S = len(lens)
    kinds = np.stack([rng.random(Tp), rng.choice(np.array([0.0, 0.125, 0.5, 2.0]), size=Tp), rng.random(Tp), np.full(Tp, 3.0)]).astype(np.float32)
    kinds[2, rng.integers(0, Tp, Tp // 50)] = np.nan
    kinds[2, rng.integers(0, Tp, Tp // 50)] = -0.0
    ctx = U.make_ctx(gen.CFG3.scaled(n_layers=L), Tp + 8, S, 16)
    a_dev = torch.from_numpy(kinds[np.arange(L) % 4]).to(U.DEV)
    for k in (1, 4096, Tp - Tp // 60, Tp):
        keep, n_keep, off, ln = _gpu_retain(U, ctx, a_dev, k, seg, S)
        for kind in range(4):
            want_keep, want_off, want_len = oracle32.retain(kinds[kind], k, seg, S)
            assert np.all(n_keep[kind::4] == len(want_keep)) and len(want_keep) == k
            assert np.all(keep[kind::4] == want_keep), (k, kind)
            assert np.all(off[kind::4] == want_off) and np.all(ln[kind::4] == want_len), (k, kind)


@pytest.mark.parametrize("Tp", [20000, 20001, 24576, 24577, 65536, 65537, 131072, 200001])
def test_retain_long_prompts(U, oracle32, Tp):
    """Several blocks per layer (from 20001 tokens on), 4096 tokens each, from 65537 tokens on 8192.  Layers: spread values; the cut among 4096 and 4097 tokens that share the first
    11 bits (the list's length, and one more: the second digit), distinct and in groups of equal ones; all tokens equal; all within one digit; mostly NaN.
    Called twice: the scratch is as the first call found it."""
    _say("retain, long prompt", Tp)
    rng = np.random.default_rng(Tp)
    lens = gen.sentence_lengths(("uniform", 1, 40), Tp + 8, seed=Tp)
    seg = np.repeat(np.arange(len(lens)), lens).astype(np.int32)
    rows = [np.exp(1.5 * rng.standard_normal(Tp))]
    for n, equal in ((4096, 1), (4097, 1), (4096, 7), (4097, 7)):
        x = np.full(Tp, 0.25)
        x[rng.permutation(Tp)[:n]] = 1.0 + (np.arange(n) // equal) * 2.0 ** -23
        rows.append(x)
    rows += [np.full(Tp, 3.0), 1.0 + rng.permutation(Tp) * 2.0 ** -21, np.where(rng.random(Tp) < 0.9, np.nan, -rng.random(Tp))]
    alpha = np.stack(rows).astype(np.float32)
    L, S = len(rows), len(lens)
    ctx = U.make_ctx(gen.CFG3.scaled(n_layers=L), Tp + 8, S, 16)
    a_dev = torch.from_numpy(alpha).to(U.DEV)
    for k in (1, 2000, 4095, 4096, 4097, Tp // 3, Tp, 2000):
        keep, n_keep, off, ln = _gpu_retain(U, ctx, a_dev, k, seg, S)
        for l in range(L):
            want_keep, want_off, want_len = oracle32.retain(alpha[l], k, seg, S)
            assert n_keep[l] == len(want_keep)
            assert np.array_equal(keep[l, :n_keep[l]], want_keep) and np.all(keep[l, n_keep[l]:] == -9), (k, l)
            assert np.array_equal(off[l], want_off) and np.array_equal(ln[l], want_len), (k, l)


@pytest.mark.parametrize("Tp", [20001, 70000, 1 << 20])
def test_retain_long_prompts_many_equal_at_the_cut(U, oracle32, Tp):
    """Equal importances at the cut, the first and the last token among them: 2 to 4096 of them in the list (up to 128 are compared with each other, more are
    ranked by the digits of their positions), and 3000 of 5000 tokens that share 22 bits, which the list does not take."""
    _say("retain, equal importances at the cut", Tp)
    rng = np.random.default_rng(Tp)
    rows = []
    for n in (4096, 3000, 1025, 129, 128, 2):
        x = np.full(Tp, 0.25)
        x[rng.permutation(np.arange(1, Tp - 1))[:n - 2]] = 1.0
        x[[0, Tp - 1]] = 1.0
        rows.append(x)
    x = np.full(Tp, 0.25)
    p = rng.permutation(Tp)
    x[p[:3000]] = 1.0
    x[p[3000:5000]] = 1.0 + rng.integers(1, 1024, 2000) * 2.0 ** -23
    rows.append(x)
    alpha = np.stack(rows).astype(np.float32)
    seg = (np.arange(Tp) // 17).astype(np.int32)
    L, S = len(rows), int(seg[-1]) + 1
    ctx = U.make_ctx(gen.CFG3.scaled(n_layers=L), Tp, S, 16)
    a_dev = torch.from_numpy(alpha).to(U.DEV)
    for k in (1, 2, 127, 128, 1024, 1025, 2999, 4095, 4999):
        keep, n_keep, off, ln = _gpu_retain(U, ctx, a_dev, k, seg, S)
        for l in range(L):
            want_keep, want_off, want_len = oracle32.retain(alpha[l], k, seg, S)
            assert n_keep[l] == len(want_keep) and np.array_equal(keep[l, :n_keep[l]], want_keep), (k, l)
            assert np.array_equal(off[l], want_off) and np.array_equal(ln[l], want_len), (k, l)


@pytest.mark.parametrize("S", [50, 3000, 7000])
def test_select_ignores_buckets_without_tokens(U, oracle32, S):
    """Zero-length buckets (a retained pool has them) are never listed, in both the register and the re-read path of
    the selection (S above 6144 takes the latter)."""
    _say("select with empty buckets, S", S)
    rng = np.random.default_rng(S)
    H = 8
    lens = rng.integers(0, 6, size=S).astype(np.int32)
    lens[rng.integers(0, S, S // 3)] = 0
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(off[-1])
    score = rng.standard_normal((H, S)).astype(np.float32)
    score[0, lens == 0] = 50.0                                        # empty buckets at the very top of a ranking
    score[1] = np.round(score[1] * 2) / 2                             # ties
    wl = gen.CFG1.scaled(n_layers=1)
    for budget in (7, 300, T + 5):
        ctx = U.make_ctx(wl, T, S, budget)
        sel = U.empty_i32(H, ctx.desc.max_sel, fill=-1)
        n_sel, n_tok = U.empty_i32(8, fill=-5), U.empty_i32(8, fill=-5)
        tok_idx = U.empty_i32(H, budget, fill=-1)
        ctx.select(torch.from_numpy(score).to(U.DEV), U.i32(off[:-1]), U.i32(lens), S, budget, sel, n_sel, tok_idx, n_tok)
        torch.cuda.synchronize()
        r_sel, r_nsel, r_tok, r_ntok = oracle32.select(score, off[:-1], lens, budget)
        g_sel, g_nsel, g_tok, g_ntok = sel.cpu().numpy(), n_sel.cpu().numpy(), tok_idx.cpu().numpy(), n_tok.cpu().numpy()
        for h in range(H):
            assert g_ntok[h] == r_ntok[h] and np.array_equal(g_tok[h, :r_ntok[h]], r_tok[h, :r_ntok[h]]), (budget, h)
            m = min(int(r_nsel[h]), ctx.desc.max_sel)
            assert g_nsel[h] == m and np.array_equal(g_sel[h, :m], r_sel[h, :m])
            assert np.all(lens[g_sel[h, :m]] > 0)


@pytest.mark.parametrize("dtype,L,k,S", [("bf16", 1, 1, 1), ("bf16", 3, 333, 97), ("bf16", 4, 6203, 2117), ("f32", 2, 5, 33), ("f32", 3, 4111, 1700)])
def test_compacted_pool_and_its_mean_keys(U, dtype, L, k, S):
    """Rows and mean keys of pools below and above the 96 MB from which values are stored past the caches, buckets of a few tokens or none, tables that end
    within a wave's buckets, a block's or at them: every layer and head at its own place."""
    _say("compacted pool", dtype, L, k, S)
    H, D, T = 8, 128, k + 1024
    rng = np.random.default_rng(k)
    wl = gen.CFG1.scaled(n_layers=L, n_tokens=T, dtype=dtype)
    ctx = U.make_ctx(wl, T, S, 1)
    g = torch.Generator(device=U.DEV)
    g.manual_seed(k)
    K, V = (torch.empty(L, H, T, D, dtype=wl.torch_dtype, device=U.DEV).normal_(generator=g) for _ in range(2))
    keep = np.stack([np.sort(rng.choice(T, k, replace=False)) for _ in range(L)]).astype(np.int32)
    off = np.sort(np.concatenate([np.zeros((L, 1), int), rng.integers(0, k + 1, (L, S - 1)), np.full((L, 1), k)], 1), 1).astype(np.int32)
    K_ret, V_ret = (torch.zeros(L, H, k, D, dtype=wl.torch_dtype, device=U.DEV) for _ in range(2))
    table = torch.full((L, H, S, D), 3.0, device=U.DEV)
    ctx.compact_pool(K, V, T, U.i32(keep), k, U.i32(np.full(L, k)), K_ret, V_ret)
    ctx.build_semvec_layers(K_ret, U.i32(off), S, table)
    torch.cuda.synchronize()
    for l in range(L):
        rows = torch.as_tensor(keep[l].astype(np.int64), device=U.DEV)
        assert torch.equal(K_ret[l], K[l].index_select(1, rows)) and torch.equal(V_ret[l], V[l].index_select(1, rows)), l
        n = np.diff(off[l])
        to = torch.as_tensor(np.repeat(np.arange(S), n), device=U.DEV)
        ref = torch.zeros(H, S, D, dtype=torch.float64, device=U.DEV).index_add_(1, to, K_ret[l].double())
        size = torch.zeros_like(ref).index_add_(1, to, K_ret[l].double().abs())
        n = torch.as_tensor(np.maximum(n, 1), device=U.DEV).view(1, S, 1)
        # n additions and a division in fp32: at most n half units in the last place of the sum of magnitudes
        assert bool(((table[l].double() - ref / n).abs() <= (n + 1) * 2.0 ** -24 * size / n).all()), l


@pytest.mark.parametrize("dtype,T,N,k,budget", [("bf16", 6000, 32, 1024, 512), ("f32", 2500, 16, 600, 256)])
def test_retention_pipeline_then_decode(U, oracle32, dtype, T, N, k, budget):
    """segment -> importance -> retain -> compact -> mean keys of the retained tokens -> fused decode step on the
    retained pool, every stage against the oracle (later stages on the GPU's retained set)."""
    _say("retention pipeline", dtype, T, N, k, budget)
    L, Hq, H, D = 2, 32, 8, 128
    wl = gen.CFG1.scaled(n_layers=L, n_tokens=T, dtype=dtype)
    p = gen.prefill_inputs(gen.CFG3.scaled(n_layers=L, n_tokens=T, dtype=dtype), seed=11, device=U.DEV)
    seg_ref, off_ref, len_ref, S = oracle32.segment(p.tok, p.bitmap, gen.CFG3.vocab)
    ctx = U.make_ctx(wl, T, S, budget)                          # tok_idx rows are max_budget wide
    seg, off, ln, S_host, _ = U.gpu_segment(ctx, p.tok, p.bitmap, gen.CFG3.vocab, S)
    assert S_host == S and np.array_equal(seg, seg_ref)
    K = p.K
    V = torch.stack([gen.kv_layer(p.lengths, H, D, wl.torch_dtype, 12, l, device=U.DEV)[1] for l in range(L)])
    q_obs = gen.queries(L * Hq, N, D, wl.torch_dtype, seed=13, device=U.DEV).view(L, Hq, N, D)
    Tp = T - N
    alpha = _gpu_importance(U, ctx, q_obs, K, T, N)
    a_np = alpha.cpu().numpy()
    keep, n_keep, r_off, r_len = _gpu_retain(U, ctx, alpha, k, seg, S)
    K_ret = torch.zeros(L, H, k, D, dtype=wl.torch_dtype, device=U.DEV)
    V_ret = torch.zeros_like(K_ret)
    ctx.compact_pool(K, V, T, U.i32(keep), k, U.i32(np.concatenate([n_keep, np.zeros(4, np.int32)])), K_ret, V_ret)
    sv = torch.full((L, H, S, D), 3.0, dtype=torch.float32, device=U.DEV)
    ctx.build_semvec_layers(K_ret, U.i32(r_off), S, sv)
    torch.cuda.synchronize()
    qd = gen.queries(L, Hq, D, wl.torch_dtype, seed=14, device=U.DEV)
    out = torch.zeros(Hq, D, dtype=torch.float32, device=U.DEV)
    tok_idx, n_tok = U.empty_i32(H, budget, fill=-1), U.empty_i32(8, fill=-5)
    n_diff = 0
    for l in range(L):
        # importance and the retained set
        a_ref = oracle32.token_importance(U.np_of(q_obs[l]), U.np_of(K[l]))
        assert np.all(np.abs(a_np[l] - a_ref) <= 2e-4 * a_ref + 1e-7 * a_ref.max())
        keep_same, off_same, len_same = oracle32.retain(a_np[l], k, seg, S)
        assert n_keep[l] == k and np.array_equal(keep[l], keep_same)
        assert np.array_equal(r_off[l], off_same) and np.array_equal(r_len[l], len_same)
        keep_e2e, _, _ = oracle32.retain(a_ref, k, seg, S)
        diff = np.setxor1d(keep_e2e, keep[l])
        if len(diff):
            cut = np.sort(a_ref)[::-1][k - 1]
            assert np.all(np.abs(a_ref[diff] - cut) <= 5e-4 * cut), (l, diff)
            n_diff += len(diff)
        assert (r_len[l] == 0).any()                              # the case does contain vanished buckets
        # compacted rows and mean keys
        Kl, Vl = U.np_of(K[l]), U.np_of(V[l])
        assert np.array_equal(U.np_of(K_ret[l]), Kl[:, keep[l]]) and np.array_equal(U.np_of(V_ret[l]), Vl[:, keep[l]])
        sv_ref = oracle32.semvec(np.ascontiguousarray(Kl[:, keep[l]])[None], r_off[l])[0]
        got = sv[l].cpu().numpy()
        kmax = float(np.abs(K[l].float().cpu().numpy()).max())
        bound = (2.0 * np.maximum(r_len[l] - 1, 0) * 2.0 ** -24 * kmax + 2.0 ** -22 * kmax)[None, :, None]
        assert np.all(np.abs(got - sv_ref) <= bound)
        assert np.all(got[:, r_len[l] == 0] == 0)
        # decode on the retained pool
        ctx.decode_step(l, 1, qd[l], qd[l], K_ret, V_ret, k, sv, S, U.i32([0, k]), U.i32([0, S]), U.i32(r_off[l]),
                        U.i32(r_len[l]), U.i32([budget]), out, None, tok_idx, n_tok)
        torch.cuda.synchronize()
        q = U.np_of(qd[l])
        ref = oracle32.decode_step(q, q, np.ascontiguousarray(Kl[:, keep[l]]), np.ascontiguousarray(Vl[:, keep[l]]), got,
                                   r_off[l][:-1], r_len[l], budget)
        g_n, g_idx = n_tok.cpu().numpy()[:H], tok_idx.cpu().numpy()
        for h in range(H):
            assert g_n[h] == ref["n_tok"][h] and np.array_equal(g_idx[h, :g_n[h]], ref["tok_idx"][h, :g_n[h]]), (l, h)
        tol = 1e-4 if dtype == "f32" else 2e-2
        assert np.abs(out.cpu().numpy() - ref["out"]).max() <= tol
    _say("  retained-set differences from the oracle's end-to-end set (documented ties):", n_diff)
