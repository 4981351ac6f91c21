"""GPU parity: every C-ABI call against the CPU oracle, element by element, on seeded
inputs.  Each call is first tested alone with oracle-made inputs (so one stage's
parity does not lean on another's), then the four calls are chained.

Bars: indices, counts, offsets and both permutation maps bit-exact; x_perm bit-exact
(a copy); routing weights 1e-5 relative; scores 1e-5 of the row's largest magnitude;
h, y_perm, y within max|gpu - ref| / max|ref| <= 2e-2 (bf16) or 1e-4 (fp32).
"""
import numpy as np
import pytest

import synth_inputs as si
from oracle import moe_oracle as orc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2603_06350_amd import binding as B  # noqa: E402
from paper_2603_06350_amd import layer  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load()


def tol_of(dtype):
    return 1e-4 if dtype == si.F32 else 2e-2


def rel_err(got, ref):
    ref = np.asarray(ref, dtype=np.float64)
    scale = np.abs(ref).max()
    return float(np.abs(np.asarray(got, dtype=np.float64) - ref).max() / (scale if scale > 0 else 1.0))


def dev(a):
    return layer.to_device(a)


def host(t):
    return layer.to_host(t)


def shape_of(cfg):
    return B.make_shape(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)


def tdtype(cfg):
    return torch.float32 if cfg.dtype == si.F32 else torch.bfloat16


# ----------------------------------------------------------------------------- route
def gpu_route(cfg, x, w_gate, bias):
    T, E, k = cfg.T, cfg.E, cfg.k
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((T, k), dtype=torch.float32, device="cuda")
    sc = torch.zeros((T, E), dtype=torch.float32, device="cuda")
    B.moe_route(shape_of(cfg), dev(x), dev(w_gate), dev(bias), idx, w, sc)
    torch.cuda.synchronize()
    return host(idx), host(w), host(sc)


def check_route(cfg, x, w_gate, bias):
    idx, w, sc = gpu_route(cfg, x, w_gate, bias)
    ridx, rw, rsc = orc.route(x, w_gate, cfg.k, cfg.renorm, bias)
    row_scale = np.maximum(np.abs(rsc).max(axis=1, keepdims=True), 1e-30)
    assert (np.abs(sc - rsc) / row_scale).max() <= 1e-5
    bad = np.nonzero((idx != ridx).any(axis=1))[0]
    assert bad.size == 0, f"{cfg.name}: top-k differs on rows {bad[:8]} gpu {idx[bad[:3]]} ref {ridx[bad[:3]]}"
    assert np.abs(w - rw).max() <= 1e-5 * max(1e-30, np.abs(rw).max())
    assert np.all(np.abs(w - rw) <= 1e-5 * np.abs(rw) + 1e-9)
    return idx, w


ROUTE_CASES = [
    dict(T=300, d=256, E=8, k=2, renorm=1),
    dict(T=1000, d=512, E=64, k=6, renorm=0),
    dict(T=77, d=1024, E=128, k=8, renorm=1),
    dict(T=130, d=264, E=200, k=5, renorm=1),     # d not a multiple of 32, E > 128
    dict(T=50, d=64, E=16, k=1, renorm=1),        # k = 1 (Llama-4-Scout style)
    dict(T=33, d=128, E=4, k=4, renorm=0),        # k = E
    dict(T=1, d=4096, E=8, k=2, renorm=1),        # one token
    dict(T=40, d=96, E=24, k=3, renorm=1, dtype=si.F32),
]


@pytest.mark.parametrize("case", ROUTE_CASES, ids=lambda c: "T{T}_d{d}_E{E}_k{k}".format(**c))
def test_route_matches_oracle(case):
    cfg = si.small_config(F=64, **case)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    check_route(cfg, L["x"], L["w_gate"], None)


def test_route_exact_ties_go_to_lowest_index():
    cfg = si.small_config(T=200, d=256, E=16, k=4, F=64)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    wg = L["w_gate"].copy()
    wg[9] = wg[2]
    wg[13] = wg[2]
    check_route(cfg, L["x"], wg, None)
    idx, w = check_route(cfg, np.zeros_like(L["x"]), wg, None)
    assert np.array_equal(idx, np.tile(np.arange(4, dtype=np.int32), (cfg.T, 1)))


def test_route_with_bias_and_forced_expert():
    cfg = si.small_config(T=150, d=256, E=64, k=6, F=64, renorm=0)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    bias = np.linspace(-2, 2, 64).astype(np.float32)
    check_route(cfg, L["x"], L["w_gate"], bias)
    bias[5] = 1e9
    bias[60:] = -1e9
    idx, _ = check_route(cfg, L["x"], L["w_gate"], bias)
    assert np.all(idx[:, 0] == 5) and idx.max() < 60


def test_route_near_ties_are_decided_like_the_oracle():
    # experts 1 and 3 share their weights and differ by a 1e-6 bias: their scores are a few
    # fp32 ulps apart, which a differently ordered fp32 sum cannot resolve but the exact pass must
    cfg = si.small_config(T=256, d=512, E=8, k=2, F=64)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    wg = L["w_gate"].copy()
    wg[3] = wg[1]
    bias = np.zeros(8, dtype=np.float32)
    bias[3] = 1e-6
    _, _, rsc = orc.route(L["x"], wg, 2, 1, bias)
    m = orc.topk_margin(rsc, 2)
    assert ((m < 1e-4) & (m > 0)).sum() > 5     # near-ties (not exact ties) at the k-th place
    check_route(cfg, L["x"], wg, bias)
    bias[3] = -1e-6
    check_route(cfg, L["x"], wg, bias)


def cancelling_tokens(T, d, E, seed):
    """bf16 inputs whose large terms cancel: the first 3/8 of a token are A*u, the next 3/8 are
    -A*u, against gate rows that repeat the same positive vector on both parts, so those products
    add up to exactly zero; the logit is what the last quarter contributes, thousands of times
    smaller than the partial sums on the way.  Experts 2i and 2i+1 differ in one element of the last
    quarter by one bf16 step: their logits are a hair apart, which is larger depends on the token,
    and every token's leading experts are such a pair."""
    rng = np.random.default_rng(seed)
    m = 3 * d // 8
    u = np.abs(rng.standard_normal((T, m), dtype=np.float32)) * 16.0
    sig = rng.standard_normal((T, d - 2 * m), dtype=np.float32) * 0.02
    x = si.f32_to_bf16_bits(np.concatenate([u, -u, sig], axis=1))
    x[:, m:2 * m] = x[:, :m] ^ np.uint16(0x8000)              # exactly the negated bf16 values
    c = np.abs(rng.standard_normal(m, dtype=np.float32)) / 16.0
    g = rng.standard_normal((E, d - 2 * m), dtype=np.float32) / 32.0
    g[1::2] = g[0::2]
    wg = si.f32_to_bf16_bits(np.concatenate([np.tile(c, (E, 1)), np.tile(c, (E, 1)), g], axis=1))
    wg[1::2, 2 * m + 5] += 1                                 # one bf16 step in one element
    return x, wg


@pytest.mark.parametrize("T,d,E,k,ws", [
    (200, 1024, 8, 2, False),      # per-tile kernel
    (2000, 1024, 8, 2, False),     # large-batch kernel, 2 tiles per block
    (3000, 1024, 64, 6, False),    # ... 64 experts
    (100, 1024, 128, 8, True),     # gate product as a kernel of its own, norms through the workspace
    (40, 2048, 256, 8, False),     # per-tile kernel, 256 experts (grouped norm tiles)
])
def test_route_when_large_terms_cancel(T, d, E, k, ws):
    """The fast pass's rounding errors follow the size of the terms it adds, not of their sum: a
    margin taken from the logits would let these tokens through with the wrong order."""
    cfg = si.small_config(T=T, d=d, E=E, k=k, F=64, renorm=1)
    x, wg = cancelling_tokens(T, d, E, seed=77)
    ridx, rw, rsc = orc.route(x, wg, k, 1, None)
    # not vacuous: the gap between experts 0 and 1 is far below what an fp32 sum of these terms
    # can resolve, and both orders occur
    gap = np.abs(rsc[:, 0] - rsc[:, 1])
    xf, wf = si.bf16_bits_to_f32(x), si.bf16_bits_to_f32(wg)
    part = np.abs(np.cumsum(xf[:8].astype(np.float64) * wf[0].astype(np.float64), axis=1)).max(axis=1)
    assert np.all(gap[:8] > 0) and np.all(gap[:8] < part * 2.0 ** -24)
    assert 0.2 < (rsc[:, 0] > rsc[:, 1]).mean() < 0.8
    if ws:
        idx, w, sc = gpu_route_ws(cfg, x, wg, None, True, True)
    else:
        idx, w, sc = gpu_route(cfg, x, wg, None)
    bad = np.nonzero((idx != ridx).any(axis=1))[0]
    assert bad.size == 0, f"top-k differs on rows {bad[:8]} gpu {idx[bad[:3]]} ref {ridx[bad[:3]]}"
    assert np.all(np.abs(w - rw) <= 1e-5 * np.abs(rw) + 1e-9)


# Batches large enough for the large-batch routing kernel (from 96 blocks of 2, 4 or 8 token tiles on;
# gate matrices of at most 128 KB take the fewest tiles per block, larger ones the most that still
# give 256 blocks; 4 or 8 tiles for 65 to 128 experts, 4 for more; k <= 16, whole 64-element stages
# per slice of the hidden dimension).  The hidden size is small so that the oracle stays fast,
# except where only a large gate matrix reaches a form.  T is never a multiple of the block.
BIG_ROUTE_CASES = [
    dict(T=8195, d=256, E=64, k=6, renorm=1),      # 2 tiles per block, 4 slices
    dict(T=8200, d=512, E=40, k=8, renorm=0),      # experts not a multiple of 16
    dict(T=8193, d=256, E=5, k=5, renorm=1),       # k = E
    dict(T=9000, d=768, E=16, k=16, renorm=0),     # the largest k this path takes, k = E
    dict(T=16400, d=256, E=16, k=1, renorm=1),     # 4 tiles per block, 2 slices
    dict(T=16390, d=384, E=33, k=3, renorm=1),
    dict(T=32800, d=128, E=8, k=2, renorm=1),
    dict(T=33000, d=64, E=64, k=15, renorm=0),     # one stage
    dict(T=32800, d=5120, E=16, k=1, renorm=0),    # 160 KB gate matrix: 8 tiles per block, up to 16 experts
    dict(T=16400, d=5120, E=16, k=2, renorm=1),    # ... 4 tiles per block
    dict(T=32800, d=2304, E=32, k=4, renorm=1),    # 8 tiles per block, up to 32 experts
    dict(T=32800, d=1088, E=64, k=6, renorm=0),    # 8 tiles per block, up to 64 experts
    dict(T=16400, d=256, E=128, k=8, renorm=1),    # more than 64 experts: 4 tiles per block only
    dict(T=16390, d=128, E=100, k=6, renorm=0),
    dict(T=16400, d=256, E=65, k=16, renorm=1),
    dict(T=32800, d=128, E=100, k=6, renorm=1),    # 8 tiles per block with more than 64 experts
    dict(T=16400, d=256, E=256, k=8, renorm=1),    # the most experts the library takes
    dict(T=16390, d=128, E=200, k=6, renorm=0),
    dict(T=3100, d=2048, E=64, k=6, renorm=1),     # 256 KB gate matrix: taken from 96 blocks on
    dict(T=6200, d=1024, E=128, k=8, renorm=0),
    dict(T=16400, d=192, E=8, k=2, renorm=1),      # slices would not be whole stages: per-tile kernel
    dict(T=8195, d=256, E=32, k=17, renorm=1),     # k too large for it: per-tile kernel
]


@pytest.mark.parametrize("case", BIG_ROUTE_CASES, ids=lambda c: "T{T}_d{d}_E{E}_k{k}".format(**c))
def test_route_large_batch_matches_oracle(case):
    cfg = si.small_config(F=64, **case)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    check_route(cfg, L["x"], L["w_gate"], None)
    bias = np.linspace(-1.5, 1.5, cfg.E).astype(np.float32)
    check_route(cfg, L["x"], L["w_gate"], bias)


@pytest.mark.parametrize("T,E", [(8195, 32), (16400, 32), (32800, 32), (16400, 128), (32800, 128),
                                 (16400, 256)])
def test_route_large_batch_ties_and_near_ties(T, E):
    # duplicated gate rows (exact ties), all-zero tokens (every score equal: more candidates than
    # the exact pass lists, so all experts are re-scored), a 1e-6 bias between two equal rows
    # (near-ties that only the exact pass resolves), experts masked by a huge negative bias
    cfg = si.small_config(T=T, d=256, E=E, k=4, F=64)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    x, wg = L["x"].copy(), L["w_gate"].copy()
    wg[9] = wg[2]
    wg[13] = wg[2]
    wg[30] = wg[17]
    x[::7] = 0
    idx, _ = check_route(cfg, x, wg, None)
    assert np.array_equal(idx[::7], np.tile(np.arange(4, dtype=np.int32), (idx[::7].shape[0], 1)))
    bias = np.zeros(E, dtype=np.float32)
    bias[13] = 1e-6
    bias[30] = -1e-6
    _, _, rsc = orc.route(x, wg, 4, 1, bias)
    m = orc.topk_margin(rsc, 4)
    assert ((m < 1e-4) & (m > 0)).sum() > 5
    check_route(cfg, x, wg, bias)
    bias[20:] = -1e9
    bias[3] = 1e9
    idx, _ = check_route(cfg, x, wg, bias)
    assert np.all(idx[:, 0] == 3) and idx.max() < 20


@pytest.mark.parametrize("T", [255, 256, 257, 300, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("dtype", [si.BF16, si.F32])
def test_route_tokens_per_block(T, dtype):
    # around the batch sizes at which a bf16 block of the per-tile kernel takes twice the tokens (up to 2049) or the
    # blocks are more than the compute units (4097)
    cfg = si.small_config(T=T, d=136, E=12, k=3, F=64, dtype=dtype)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    check_route(cfg, L["x"], L["w_gate"], None)


@pytest.mark.parametrize("T,d,E", [(1000, 136, 12), (2047, 136, 12), (8191, 32, 48), (2000, 1024, 16), (513, 16, 129),
                                   (1023, 2048, 129), (4095, 16, 256), (511, 1024, 128), (2047, 1024, 128)])
def test_route_fp32_several_tokens_per_block(T, d, E):
    # 2, 4, 16 and 2 tokens per block of layers with a small gate, 1 (three rounds), 4 and 16 with more than 128 experts,
    # 2 and 8 with a large gate; the last block is short
    cfg = si.small_config(T=T, d=d, E=E, k=3, F=64, dtype=si.F32)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    check_route(cfg, L["x"], L["w_gate"], None)


@pytest.mark.parametrize("d", [2048, 2560, 4096, 5120, 8192])
@pytest.mark.parametrize("near", [2, 3])
def test_route_equal_gate_rows_get_equal_exact_scores(d, near):
    # `near` tokens of every 32-token block go through the exact pass with all 12 experts: 24 or 36 pairs, so a
    # token's pairs are split between a group of 16, 8 or 4 and a shorter one.  Their large terms cancel, and the sums of
    # such terms depend on their order even in fp64: the equal rows 3 and 5 have to be summed in one order.
    T, E, k, A = 4096, 12, 4, 2.0 ** 30
    rng = np.random.default_rng(d)
    w = rng.standard_normal((E, d))
    w[:, 0:d // 2:2] = np.abs(w[:, 0:d // 2:2]) + 0.5
    w[:, d // 2::2] = w[:, 0:d // 2:2]
    w[5] = w[3]
    x = rng.standard_normal((T, d))
    x -= np.outer(x @ w[3] / (w[3] @ w[3]) + 8.0 / np.sqrt(w[3] @ w[3]), w[3])    # (3 and 5 last for all other tokens)
    large = np.arange(T) % 32 < near
    u = A * rng.uniform(0.5, 2.0, size=(int(large.sum()), d // 4))
    half = x[large]
    half[:, 0:d // 2:2], half[:, d // 2::2] = u, -u
    x[large] = half
    cfg = si.small_config(T=T, d=d, E=E, k=k, F=64)
    idx, _, sc = gpu_route(cfg, si.f32_to_bf16_bits(x.astype(np.float32)), si.f32_to_bf16_bits(w.astype(np.float32)), None)
    assert np.array_equal(sc[:, 3].view(np.int32), sc[:, 5].view(np.int32))
    at = np.where(idx == 3, np.arange(k), k).min(axis=1)
    assert np.all(np.where(idx == 5, np.arange(k), k).min(axis=1) >= np.minimum(at + 1, k))


def test_route_fp32_batch_too_large_for_a_block_per_token():
    # 2^23 blocks of 512 threads are one more than a launch takes
    T, d, E = 2 ** 23 + 3, 4, 3
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn((T, d), device="cuda", generator=gen)
    w = torch.randn((E, d), device="cuda", generator=gen)
    idx = torch.full((T, 1), -1, dtype=torch.int32, device="cuda")
    weight = torch.zeros((T, 1), device="cuda")
    B.moe_route(B.make_shape(T, d, E, 1, 64, si.F32, 0), x, w, None, idx, weight)
    torch.cuda.synchronize()
    score = (x.double()[:, None, :] * w.double()[None]).sum(dim=2).float()   # (products exact, one rounding)
    want = score.argmax(dim=1)
    best = score.gather(1, want[:, None])
    assert bool(((idx[:, 0] == want) | (score.gather(1, idx.long()) == best)[:, 0]).all())
    assert bool(((weight - torch.softmax(score, dim=1).gather(1, want[:, None])).abs() <= 1e-5).all())


@pytest.mark.parametrize("d", [1024, 4096, 5120, 16384])
def test_route_few_near_ties_per_block(d):
    # 0 to 11 tokens of every 32-token block have two equal scores beside chosen ones up to a bias that only the
    # exact pass sees: 0 to 22 (token, expert) pairs per block, summed 16, 8 or 4 at a time (wider rows, fewer)
    cfg = si.small_config(T=3100, d=d, E=8, k=2, F=64)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    wg = L["w_gate"].copy()
    wg[5] = wg[3]
    w3 = si.bf16_bits_to_f32(wg[3]).astype(np.float64)
    x = si.bf16_bits_to_f32(L["x"]).astype(np.float64)
    x -= np.outer(x @ w3 / (w3 @ w3), w3)             # experts 3 and 5 score 0 ...
    t = np.arange(cfg.T)
    near = t % 32 < (t // 32) % 12
    x += np.outer(np.where(near, 8.0, -8.0), w3 / np.sqrt(w3 @ w3))   # ... then far above or far below the others
    x = si.f32_to_bf16_bits(x.astype(np.float32))
    bias = np.zeros(cfg.E, dtype=np.float32)
    bias[5] = 1e-6
    idx, _ = check_route(cfg, x, wg, bias)
    pair = np.isin(idx, (3, 5)).sum(axis=1)
    assert (pair[near] == 2).mean() > 0.9 and pair[~near].max() == 0


def test_route_large_batch_without_scores_output():
    cfg = si.small_config(T=8200, d=256, E=64, k=6, F=64)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    idx = torch.full((cfg.T, cfg.k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((cfg.T, cfg.k), dtype=torch.float32, device="cuda")
    B.moe_route(shape_of(cfg), dev(L["x"]), dev(L["w_gate"]), None, idx, w, None)
    torch.cuda.synchronize()
    ridx, rw, _ = orc.route(L["x"], L["w_gate"], cfg.k, cfg.renorm, None)
    assert np.array_equal(host(idx), ridx)
    assert np.all(np.abs(host(w) - rw) <= 1e-5 * np.abs(rw) + 1e-9)


# Small batches with a gate matrix of at least 256 KB: with a workspace (or a score output) the
# gate product runs as a kernel of its own over the whole chip and the selection reads its scores.
SMALL_ROUTE_WS_CASES = [
    dict(T=32, d=4096, E=128, k=8, renorm=1),      # the decode-shaped layer's routing
    dict(T=77, d=1024, E=128, k=8, renorm=0),      # exactly 256 KB
    dict(T=130, d=2056, E=200, k=5, renorm=1),     # ragged hidden size, E > 128, E % 16 != 0
    dict(T=512, d=2048, E=64, k=6, renorm=1),
    dict(T=2048, d=1024, E=128, k=8, renorm=1),    # enough token tiles for 64-expert gate tiles
    dict(T=3000, d=520, E=256, k=8, renorm=0),     # more than 128 experts, ragged hidden size
    dict(T=1, d=4096, E=33, k=33, renorm=1),       # one token, k = E
]


def gpu_route_ws(cfg, x, w_gate, bias, with_ws, with_scores):
    T, E, k = cfg.T, cfg.E, cfg.k
    sh = shape_of(cfg)
    idx = torch.full((T, k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((T, k), dtype=torch.float32, device="cuda")
    sc = torch.full((T, E), -3.0, dtype=torch.float32, device="cuda") if with_scores else None
    nb = B.moe_workspace_bytes(sh)
    assert nb >= T * E * 4 or T >= 8192     # room for the scores of every batch that can use them
    ws = torch.full((nb,), 0x5A, dtype=torch.uint8, device="cuda") if with_ws else None
    B.moe_route_ws(sh, dev(x), dev(w_gate), dev(bias), idx, w, sc, ws, nb if with_ws else 0)
    torch.cuda.synchronize()
    return host(idx), host(w), (host(sc) if with_scores else None)


@pytest.mark.parametrize("case", SMALL_ROUTE_WS_CASES, ids=lambda c: "T{T}_d{d}_E{E}_k{k}".format(**c))
def test_route_with_workspace_matches_oracle_and_plain_route(case):
    cfg = si.small_config(F=64, **case)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    x, wg = L["x"].copy(), L["w_gate"].copy()
    wg[cfg.E - 1] = wg[0]                           # an exact tie between the first and the last expert
    x[cfg.T // 2] = 0                               # and a token whose scores are all equal
    bias = np.linspace(-1.0, 1.0, cfg.E).astype(np.float32)
    for b in (None, bias):
        ridx, rw, rsc = orc.route(x, wg, cfg.k, cfg.renorm, b)
        pidx, pw, psc = gpu_route(cfg, x, wg, b)    # moe_route: one kernel
        assert np.array_equal(pidx, ridx)
        for with_ws, with_scores in ((True, False), (False, True), (True, True)):
            idx, w, sc = gpu_route_ws(cfg, x, wg, b, with_ws, with_scores)
            assert np.array_equal(idx, ridx), (with_ws, with_scores)
            assert np.all(np.abs(w - rw) <= 1e-5 * np.abs(rw) + 1e-9)
            # the two forms take the choice on the same fast scores and re-score near-ties exactly;
            # which tokens count as near-ties may differ in the last bits of the margin, so weights
            # and scores agree to the oracle's tolerance rather than bit for bit
            assert np.all(np.abs(w - pw) <= 1e-5 * np.abs(pw) + 1e-9)
            if with_scores:
                assert np.all(np.abs(sc - psc) <= 1e-5 * np.abs(psc).max(axis=1, keepdims=True))


def test_route_ws_without_usable_workspace_is_plain_route():
    cfg = si.small_config(T=32, d=4096, E=128, k=8, F=64)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    ridx, rw, _ = orc.route(L["x"], L["w_gate"], cfg.k, cfg.renorm, None)
    idx = torch.full((cfg.T, cfg.k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((cfg.T, cfg.k), dtype=torch.float32, device="cuda")
    small = torch.zeros((256,), dtype=torch.uint8, device="cuda")       # too small: ignored
    B.moe_route_ws(shape_of(cfg), dev(L["x"]), dev(L["w_gate"]), None, idx, w, None, small, 256)
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ridx)
    assert np.all(np.abs(host(w) - rw) <= 1e-5 * np.abs(rw) + 1e-9)


def test_route_ws_with_room_for_the_scores_but_not_the_norms_is_plain_route():
    # the two-kernel form needs T*E scores and T + E norms: a workspace of exactly T*E*4 bytes is
    # not enough for it, and the call must behave like moe_route
    cfg = si.small_config(T=48, d=2048, E=128, k=8, F=64)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    ridx, rw, _ = orc.route(L["x"], L["w_gate"], cfg.k, cfg.renorm, None)
    idx = torch.full((cfg.T, cfg.k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((cfg.T, cfg.k), dtype=torch.float32, device="cuda")
    nb = cfg.T * cfg.E * 4
    ws = torch.full((nb + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    B.moe_route_ws(shape_of(cfg), dev(L["x"]), dev(L["w_gate"]), None, idx, w, None, ws, nb)
    torch.cuda.synchronize()
    assert np.array_equal(host(idx), ridx)
    assert np.all(np.abs(host(w) - rw) <= 1e-5 * np.abs(rw) + 1e-9)
    assert bool((ws[nb:] == 0x5A).all())            # nothing written past the size it was given


# ----------------------------------------------------------------------------- count + permute
def gpu_dispatch(cfg, x, idx):
    T, E, k, d = cfg.T, cfg.E, cfg.k, cfg.d
    sh = shape_of(cfg)
    A = T * k
    counts = torch.full((E,), -7, dtype=torch.int32, device="cuda")
    offsets = torch.full((E + 1,), -7, dtype=torch.int32, device="cuda")
    dst = torch.full((max(A, 1),), -7, dtype=torch.int32, device="cuda")
    src = torch.full((max(A, 1),), -7, dtype=torch.int32, device="cuda")
    xp = torch.zeros((max(A, 1), d), dtype=tdtype(cfg), device="cuda")
    nb = B.moe_workspace_bytes(sh)
    ws = torch.full((nb,), 0x5A, dtype=torch.uint8, device="cuda")   # garbage on entry
    B.moe_count_and_permute(sh, dev(x), dev(idx), counts, offsets, dst, src, xp, ws, nb)
    torch.cuda.synchronize()
    return host(counts), host(offsets), host(dst)[:A], host(src)[:A], host(xp)[:A]


def check_dispatch(cfg, x, idx):
    counts, offsets, dst, src, xp = gpu_dispatch(cfg, x, idx)
    rc, ro = orc.expert_load(idx, cfg.E)
    rd, rs = orc.permutation(idx, cfg.E)
    assert np.array_equal(counts, rc)
    assert np.array_equal(offsets, ro)
    assert np.array_equal(dst, rd)
    assert np.array_equal(src, rs)
    assert np.array_equal(xp, orc.permute_rows(x, rd, cfg.k))
    assert counts.sum() == cfg.T * cfg.k


DISPATCH_CASES = [
    dict(T=300, d=256, E=8, k=2),
    dict(T=1000, d=128, E=64, k=6),       # several blocks of 256 tokens, ragged tail
    dict(T=513, d=64, E=128, k=8),
    dict(T=700, d=72, E=256, k=3),        # 128-thread variant, row not a multiple of 64 B
    dict(T=1, d=4096, E=8, k=2),
    dict(T=40, d=96, E=24, k=3, dtype=si.F32),
    dict(T=128, d=64, E=16, k=2),         # 256 assignments: the largest single-launch dispatch
    dict(T=512, d=64, E=16, k=2),         # 1024 assignments: two launches
    dict(T=86, d=64, E=16, k=3),          # 258: the smallest that takes the general path
    dict(T=32, d=64, E=256, k=8),         # single launch, most experts
]


@pytest.mark.parametrize("case", DISPATCH_CASES, ids=lambda c: "T{T}_d{d}_E{E}_k{k}".format(**c))
def test_count_and_permute_matches_oracle(case):
    cfg = si.small_config(F=64, **case)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    idx, _, _ = orc.route(L["x"], L["w_gate"], cfg.k, cfg.renorm)
    check_dispatch(cfg, L["x"], idx)


def test_count_and_permute_degenerate_loads():
    cfg = si.small_config(T=600, d=64, E=16, k=2, F=64)
    L = si.make_layer(cfg, parts=("x",))
    idx = np.zeros((cfg.T, 2), dtype=np.int32)
    idx[:, 0], idx[:, 1] = 7, 3                       # two experts take everything, 14 are empty
    check_dispatch(cfg, L["x"], idx)
    rng = np.random.default_rng(0)
    idx = rng.integers(0, 16, size=(cfg.T, 2)).astype(np.int32)   # a token may repeat an expert
    check_dispatch(cfg, L["x"], idx)
    cfg1 = si.small_config(T=600, d=64, E=16, k=1, F=64)
    check_dispatch(cfg1, L["x"], np.full((cfg.T, 1), 15, dtype=np.int32))
    # the same degenerate loads in a batch small enough for the single-launch dispatch
    cfg2 = si.small_config(T=120, d=64, E=16, k=2, F=64)
    L2 = si.make_layer(cfg2, parts=("x",))
    idx = np.zeros((cfg2.T, 2), dtype=np.int32)
    idx[:, 0], idx[:, 1] = 7, 3
    check_dispatch(cfg2, L2["x"], idx)
    idx = np.random.default_rng(1).integers(0, 16, size=(cfg2.T, 2)).astype(np.int32)   # repeats
    check_dispatch(cfg2, L2["x"], idx)


@pytest.mark.parametrize("T,d,E,k", [(1, 64, 1, 1), (255, 72, 3, 1), (64, 520, 5, 4), (257, 64, 65, 1), (512, 1032, 256, 2),
                                     (6143, 64, 9, 1), (1536, 64, 256, 4), (6145, 64, 9, 1), (1537, 64, 256, 4)])
def test_count_and_permute_on_both_sides_of_the_single_launch_limit(T, d, E, k):
    """Batches of up to 6144 assignments are ranked by counting smaller keys, larger ones by histogram
    and scan: the largest and smallest of each, blocks of 256 keys and 512-element rows over- and underfilled."""
    cfg = si.small_config(T=T, d=d, E=E, k=k, F=64)
    L = si.make_layer(cfg, parts=("x",))
    idx = np.random.default_rng(T + E).integers(0, E, size=(T, k)).astype(np.int32)
    check_dispatch(cfg, L["x"], idx)


@pytest.mark.parametrize("T", [2816, 6145, 20001])
@pytest.mark.parametrize("E,k", [(1, 1), (3, 3), (7, 7), (17, 8), (64, 9), (128, 16), (129, 24), (256, 5)])
def test_count_and_permute_two_launches_by_experts_and_choices(T, E, k):
    # up to eight choices per token stay in registers, more are read again; tables of experts that divide a block's
    # threads or not; blocks with one token, and partial counts of one batch of loads and several
    cfg = si.small_config(T=max(T, 6145 // k + 1), d=16, E=E, k=k, F=64)
    L = si.make_layer(cfg, parts=("x",))
    idx = np.random.default_rng(T + E).integers(0, E, size=(cfg.T, k)).astype(np.int32)
    check_dispatch(cfg, L["x"], idx)


@pytest.mark.parametrize("chunks", [1, 63, 255, 256, 257, 520])
@pytest.mark.parametrize("E", [7, 24, 25])
def test_count_and_permute_row_copy_at_the_edges_of_its_steps(E, chunks):
    # above 6144 assignments a wave copies 256 chunks of 16 bytes of a token's row per step; with up to 256
    # rows per expert (E = 25: 252, 24: 262) the stores are streamed
    cfg = si.small_config(T=2100, d=chunks * 8, E=E, k=3, F=64)
    L = si.make_layer(cfg, parts=("x",))
    check_dispatch(cfg, L["x"], np.random.default_rng(chunks).integers(0, E, size=(cfg.T, 3)).astype(np.int32))


@pytest.mark.parametrize("T", [32768, 32769, 65536, 65537, 100001])
def test_count_and_permute_row_copy_around_the_size_of_the_memory_side_cache(T):
    # x and x_perm of 256 MiB together, where the stores turn to streaming, x of 256 MiB alone, where the
    # loads do, and past it
    d, E = 2048, 5
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.empty((T, d), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    idx = torch.randint(0, E, (T, 1), dtype=torch.int32, device="cuda", generator=gen)
    counts, offsets, dst, src = (torch.zeros(n, dtype=torch.int32, device="cuda") for n in (E, E + 1, T, T))
    x_perm = torch.zeros_like(x)
    sh = B.make_shape(T, d, E, 1, 64, si.BF16, 1)
    nb = B.moe_workspace_bytes(sh)
    ws = torch.empty((nb,), dtype=torch.uint8, device="cuda")
    B.moe_count_and_permute(sh, x, idx, counts, offsets, dst, src, x_perm, ws, nb)
    torch.cuda.synchronize()
    order = torch.sort(idx[:, 0].long(), stable=True).indices
    assert torch.equal(src.long(), order) and torch.equal(x_perm, x[order])


def test_count_and_permute_leaves_invalid_experts_out():
    cfg = si.small_config(T=301, d=64, E=6, k=2, F=64)
    idx = np.random.default_rng(2).integers(0, 6, size=(cfg.T, 2)).astype(np.int32)
    idx[5, 0], idx[299, 1] = -1, 6
    sh, flat = shape_of(cfg), idx.reshape(-1)
    A = flat.size
    out = [torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (6, 7, A, A)]
    nb = B.moe_workspace_bytes(sh)
    ws = torch.empty((nb,), dtype=torch.uint8, device="cuda")
    B.moe_count_and_permute(sh, None, dev(idx), *out, None, ws, nb)
    torch.cuda.synchronize()
    counts, offsets, dst, src = (host(o) for o in out)
    valid = (flat >= 0) & (flat < 6)
    order = np.flatnonzero(valid)[np.argsort(flat[valid], kind="stable")]
    assert np.array_equal(counts, np.bincount(flat[valid], minlength=6))
    assert np.array_equal(offsets, np.concatenate([[0], np.cumsum(counts)]))
    assert np.array_equal(src[:order.size], order) and np.array_equal(dst[order], np.arange(order.size))
    assert ((dst >= 0) & (dst < A)).all()


def test_count_and_permute_no_tokens():
    cfg = si.small_config(T=0, d=64, E=8, k=2, F=64)
    sh = shape_of(cfg)
    counts = torch.full((8,), -7, dtype=torch.int32, device="cuda")
    offsets = torch.full((9,), -7, dtype=torch.int32, device="cuda")
    nb = B.moe_workspace_bytes(sh)
    ws = torch.empty((nb,), dtype=torch.uint8, device="cuda")
    B.moe_count_and_permute(sh, None, None, counts, offsets, None, None, None, ws, nb)
    torch.cuda.synchronize()
    assert host(counts).tolist() == [0] * 8 and host(offsets).tolist() == [0] * 9


# ----------------------------------------------------------------------------- grouped FFN
def gpu_ffn(cfg, x_perm, offsets, w1, w3, w2):
    A = cfg.T * cfg.k
    h = torch.zeros((A, cfg.F), dtype=tdtype(cfg), device="cuda")
    yp = torch.zeros((A, cfg.d), dtype=tdtype(cfg), device="cuda")
    args = (dev(x_perm), None, dev(offsets), dev(w1), dev(w3), dev(w2))
    B.moe_grouped_ffn(shape_of(cfg), args[0], *args[2:], h, yp)
    # Inputs this small leave the last (only) round of tiles under-filled, so the call above cuts
    # its tiles along the rows into pieces; with 4 added to `parts` every tile stays whole, which is
    # how the tiles of a full-size batch run.  Both forms are checked: same bits, and the caller
    # compares them with the oracle.
    h_whole, yp_whole = torch.zeros_like(h), torch.zeros_like(yp)
    B.moe_grouped_ffn_ws(shape_of(cfg), *args, h_whole, yp_whole, 3 | 4, None, 0)
    torch.cuda.synchronize()
    assert torch.equal(h, h_whole), "h differs between cut and whole tiles"
    assert torch.equal(yp, yp_whole), "y_perm differs between cut and whole tiles"
    return orc.to_f64(host(h)), orc.to_f64(host(yp))


def check_ffn(cfg, L, idx):
    _, offsets = orc.expert_load(idx, cfg.E)
    dst, _ = orc.permutation(idx, cfg.E)
    x_perm = orc.permute_rows(L["x"], dst, cfg.k)
    ry, rh = orc.grouped_ffn(x_perm, offsets, L["w1"], L["w3"], L["w2"], return_h=True)
    h, yp = gpu_ffn(cfg, x_perm, offsets, L["w1"], L["w3"], L["w2"])
    tol = tol_of(cfg.dtype)
    assert rel_err(h, rh) <= tol, f"h: {rel_err(h, rh):.3e}"
    assert rel_err(yp, ry) <= tol, f"y_perm: {rel_err(yp, ry):.3e}"
    # per-row check too: a wrong row hiding behind a large global scale would show here
    row_scale = np.abs(ry).max(axis=1) + 1e-30
    assert (np.abs(yp - ry).max(axis=1) / row_scale).max() <= 4 * tol
    return x_perm, offsets, dst


FFN_CASES = [
    dict(T=300, d=256, E=8, k=2, F=384),          # 75 rows/expert: tiles of up to 128 rows
    dict(T=600, d=256, E=8, k=2, F=384),          # 150 rows/expert: one tile per expert
    dict(T=1500, d=128, E=2, k=1, F=256),         # 750 rows/expert: three tiles per expert
    dict(T=900, d=192, E=3, k=2, F=320),          # 600 rows/expert, N tails (320 = 2.5 x 128, 192 < 256)
    dict(T=64, d=512, E=64, k=6, F=128),          # many small / empty experts
    dict(T=100, d=200, E=4, k=2, F=104),          # d, F not multiples of 64
    dict(T=64, d=128, E=8, k=2, F=256, dtype=si.F32, x_std=0.02, w_std=0.02),
    dict(T=45, d=36, E=5, k=2, F=52, dtype=si.F32),
]


def test_grouped_ffn_few_rows_per_expert_with_one_hot_expert():
    # few rows per expert on average (tiles of up to 128 rows), but one expert holds several tiles'
    # worth of rows and most are empty
    cfg = si.small_config(T=400, d=256, E=64, k=1, F=384)
    L = si.make_layer(cfg)
    rng = np.random.default_rng(5)
    idx = np.where(rng.random((cfg.T, 1)) < 0.8, 5, rng.integers(0, 64, size=(cfg.T, 1))).astype(np.int32)
    counts, _ = orc.expert_load(idx, cfg.E)
    assert counts[5] > 4 * 64 and (counts == 0).sum() > 10
    check_ffn(cfg, L, idx)


@pytest.mark.parametrize("case", FFN_CASES, ids=lambda c: "T{T}_d{d}_E{E}_k{k}_F{F}".format(**c))
def test_grouped_ffn_matches_oracle(case):
    cfg = si.small_config(**case)
    L = si.make_layer(cfg)
    idx, _, _ = orc.route(L["x"], L["w_gate"], cfg.k, cfg.renorm)
    check_ffn(cfg, L, idx)


@pytest.mark.parametrize("d,F", [(64, 704), (128, 640), (192, 576), (256, 512), (320, 448), (384, 384)])
def test_grouped_ffn_every_stage_count_of_the_two_stage_pipeline(d, F):
    # K stages of 64 elements: the up-projection takes d / 64 of them and the down-projection F / 64,
    # so the six cases run the even tiles' two-buffer pipeline over 1 to 11 stages (prologue only,
    # odd and even counts); the experts hold one tile of 256 rows (every wave four sub-tiles), one of
    # 300 rows (19 sub-tiles: waves with five and with four) and two tiles of 224 rows (waves with
    # four and with three sub-tiles)
    cfg = si.small_config(T=1000, d=d, E=3, k=1, F=F)
    L = si.make_layer(cfg)
    idx = np.zeros((cfg.T, 1), dtype=np.int32)
    idx[:256] = 0
    idx[256:256 + 300] = 1
    idx[556:] = 2
    check_ffn(cfg, L, idx)


@pytest.mark.parametrize("d,F", [(8, 8), (16, 120), (56, 72), (64, 136), (72, 64), (136, 264), (248, 1032), (520, 392)])
@pytest.mark.parametrize("T,E", [(37, 5), (1000, 3), (1700, 11)])
def test_grouped_ffn_widths_that_are_multiples_of_8(T, E, d, F):
    # K tails of 1 to 7 chunks (also a single, partial stage), N tails of one row group up to one
    # short of a tile; ring tiles (7 rows per expert), even tiles (154 and 333), ragged last sub-tiles
    cfg = si.small_config(T=T, d=d, E=E, k=1, F=F, seed=d + F)
    L = si.make_layer(cfg)
    idx = np.random.default_rng(T).integers(0, E, size=(T, 1)).astype(np.int32)
    if T == 1000:
        idx[:400] = 0                             # tiles of 304 and of 320 rows and more
    check_ffn(cfg, L, idx)


@pytest.mark.parametrize("rows", [40, 100, 300])
def test_grouped_ffn_extreme_gates_at_widths_that_are_multiples_of_8(rows):
    # finite gates whose product with the up value, or whose exponential, leaves the fp32 range: silu is
    # taken before the product, by a true division (ring tiles, and even tiles of 100 and 300 rows)
    d, F = 72, 136
    cfg = si.small_config(T=rows, d=d, E=1, k=1, F=F)
    L = si.make_layer(cfg)
    f32 = lambda a: (a.astype(np.uint32) << 16).view(np.float32)
    bits = lambda a: (np.ascontiguousarray(a, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
    x, w1, w3 = (f32(L[n]).copy() for n in ("x", "w1", "w3"))
    x[:, 0], x[:, 1] = 1.0, 0.0
    gates = np.array([-1e20, 1e18, -1e38, -200.0, -104.0, -88.0, -86.5, -60.0], np.float32)
    ups = np.array([1e20, 1e18, -1e38, 2e38, 1e38, 2.0 ** 100, -2.0 ** 110, 2.0 ** 90], np.float32)
    w1[0, :8], w3[0, :8] = 0.0, 0.0               # these eight columns: gate and up value are the constants above
    w1[0, :8, 0], w3[0, :8, 0] = gates, ups
    x, w1, w3 = bits(x), bits(w1), bits(w3)
    offsets = np.array([0, rows], np.int32)
    h = torch.zeros((rows, F), dtype=torch.bfloat16, device="cuda")
    yp = torch.zeros((rows, d), dtype=torch.bfloat16, device="cuda")
    B.moe_grouped_ffn(shape_of(cfg), dev(x), dev(offsets), dev(w1), dev(w3), dev(L["w2"]), h, yp)
    torch.cuda.synchronize()
    g, u = f32(w1[0, :8, 0]).astype(np.float64), f32(w3[0, :8, 0]).astype(np.float64)
    want = np.array([a * b / (1.0 + np.exp(-a)) if a > -700.0 else 0.0 for a, b in zip(g, u)])
    got = h[:, :8].float().cpu().numpy().astype(np.float64)
    # beyond exp(-g) = inf in fp32 (g below -88.7) silu is 0; else a few fp32 roundings and one to bf16 (2^-9)
    want[g < -88.7] = 0.0
    assert np.isfinite(got).all()
    assert (np.abs(got - want) <= 2.0 ** -8 * np.abs(want)).all(), (got[0], want)


@pytest.mark.parametrize("d,F", [(4, 4), (28, 60), (32, 64), (36, 68), (64, 132), (136, 100)])
@pytest.mark.parametrize("rows", [(1, 0, 33), (16, 17, 31, 32), (64, 65, 129, 5)])
def test_grouped_ffn_fp32_tile_edges(rows, d, F):
    # K tails of 1 to 7 chunks of four, N tails around the 64 weight rows of a tile, rows around the
    # 16-row sub-tiles and the 32-row tiles; the last case's down-projection also in 64-row tiles below
    cfg = si.small_config(T=sum(rows), d=d, E=len(rows), k=1, F=F, dtype=si.F32, seed=d + F + rows[0])
    check_ffn(cfg, si.make_layer(cfg), np.repeat(np.arange(len(rows), dtype=np.int32), rows)[:, None])


def test_grouped_ffn_fp32_64_row_tiles():
    # enough tiles (16 per compute unit) for the 64-row form of both GEMMs, segments of every row count
    # modulo 64 that is near an edge
    rows = (2000, 2049, 2063, 2064, 2111, 63)
    cfg = si.small_config(T=sum(rows), d=1608, E=len(rows), k=1, F=1612, dtype=si.F32)
    L = si.make_layer(cfg)
    idx = np.repeat(np.arange(len(rows), dtype=np.int32), rows)[:, None]
    counts, offsets = orc.expert_load(idx, cfg.E)     # (token order is already the permuted order)
    h, yp = gpu_ffn(cfg, L["x"], offsets, L["w1"], L["w3"], L["w2"])
    at = np.unique(np.concatenate([np.r_[o:min(o + 70, o + n), max(o, o + n - 70):o + n]
                                   for o, n in zip(offsets[:-1], counts)]))
    ry, rh = orc.grouped_ffn(L["x"][at], np.searchsorted(at, offsets), L["w1"], L["w3"], L["w2"], return_h=True)
    assert rel_err(h[at], rh) <= tol_of(cfg.dtype) and rel_err(yp[at], ry) <= tol_of(cfg.dtype)
    assert np.isfinite(h).all() and np.isfinite(yp).all()


def two_norm_err(got, ref):
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("d,F", [(2052, 2076), (2080, 2064), (2076, 2080)])
@pytest.mark.parametrize("rows", [(33, 64, 112, 0, 128, 48, 127, 128), (65, 64, 129, 3, 200, 40, 150, 32)], ids=["split", "mixed"])
def test_grouped_ffn_fp32_split_tiles(rows, d, F):
    # 64-row tiles in three bf16 pieces per value (36 rows per expert and more than 5/4 tiles per CU in both GEMMs): tiles of
    # 33, 48 and 64 rows, in the second list also of up to 32, which take the fp32 instruction; K tails of 1, 4
    # and 7 chunks, whole stages, N tails.  Bounds, 2-norm against 64-bit sums: the pieces' error is 4.8e-7 at these
    # widths, the fp32 instruction's 1.25e-6 (the matrix instructions do not round to nearest, so it grows with
    # K), and a missing second-order piece product is 3.5e-6 on either GEMM.
    cfg = si.small_config(T=sum(rows), d=d, E=len(rows), k=1, F=F, dtype=si.F32, seed=d)
    L = si.make_layer(cfg)
    idx = np.repeat(np.arange(len(rows), dtype=np.int32), rows)[:, None]
    _, offsets = orc.expert_load(idx, cfg.E)          # (token order is already the permuted order)
    h, yp = gpu_ffn(cfg, L["x"], offsets, L["w1"], L["w3"], L["w2"])
    ry, rh = orc.grouped_ffn(L["x"], offsets, L["w1"], L["w3"], L["w2"], return_h=True)
    bound = 1e-6 if min(n % 64 == 0 or n % 64 > 32 for n in rows if n) else 2e-6
    assert two_norm_err(h, rh) <= bound
    own = np.concatenate([h[a:b] @ L["w2"][e].astype(np.float64).T for e, (a, b) in enumerate(zip(offsets[:-1], offsets[1:]))])
    assert two_norm_err(yp, own) <= bound             # (of the GPU's own h: the second GEMM's error alone)
    assert rel_err(yp, ry) <= tol_of(cfg.dtype)
    for e, (a, b) in enumerate(zip(offsets[:-1], offsets[1:])):   # (a tile or a sub-tile of its own must not hide)
        for r in range(a, b, 16):
            assert two_norm_err(h[r:min(r + 16, b)], rh[r:min(r + 16, b)]) <= 2e-6, (e, r)
            assert two_norm_err(yp[r:min(r + 16, b)], own[r:min(r + 16, b)]) <= 2e-6, (e, r)


# (exponent of the row's value, of the weights, of further values in the same rows that meet zeros only)
ONE_TERM = [(0, 0, None), (0, 0, 60), (-115, 20, 30), (20, -115, 40), (-60, -60, None), (-60, -58, 50), (39, 38, None)]


@pytest.mark.parametrize("ex,ew,big", ONE_TERM)
@pytest.mark.parametrize("part", [1, 2])
@pytest.mark.parametrize("at", [1, 70])
def test_grouped_ffn_fp32_split_tiles_sums_of_one_product(part, at, ex, ew, big):
    # every sum is one product, so each of the eight piece products (the smallest are 2^-25 of the whole) shows in the
    # result: the rounded product, within 2^-24 and what the pieces' own sum adds (2^-31).  Values near the lower end of
    # fp32, also beside values that are far larger.  A missing product of order 2^-25 gives 1.2 x 2^-24 and more.
    K, N, rows = 100, 64 * 322, 64
    gen = torch.Generator(device="cuda").manual_seed(11)
    v = (torch.rand(rows, device="cuda", generator=gen) + 1.0) * 2.0 ** ex
    w = (torch.rand(N, device="cuda", generator=gen) + 1.0) * 2.0 ** ew
    a, b = torch.zeros((rows, K), device="cuda"), torch.zeros((N, K), device="cuda")
    a[:, at], b[:, at] = v, w
    if big is not None:
        a[:, 50], b[:, 51] = 2.0 ** big, 2.0 ** big
    off = torch.tensor([0, rows], dtype=torch.int32, device="cuda")
    if part == 1:                                     # gate values of 128: silu(128) is 128 in fp32
        a[:, 0] = 1.0
        gate = torch.zeros_like(b)
        gate[:, 0] = 128.0
        out, other = torch.zeros((rows, N), device="cuda"), torch.zeros((rows, K), device="cuda")
        B.moe_grouped_ffn_part(B.make_shape(rows, K, 1, 1, N, si.F32, 1), a, off, gate[None], b[None],
                               torch.zeros((1, K, N), device="cuda"), out, other, 1)
        out = out / 128.0
    else:
        out, other = torch.zeros((rows, N), device="cuda"), torch.zeros((1, K, N), device="cuda")
        B.moe_grouped_ffn_part(B.make_shape(rows, N, 1, 1, K, si.F32, 1), torch.zeros((rows, N), device="cuda"), off,
                               torch.zeros((1, K, N), device="cuda"), other, b[None], a, out, 2)
    torch.cuda.synchronize()
    want = v.double()[:, None] * w.double()[None]
    assert float(((out.double() - want).abs() / want).max()) <= 2.0 ** -24 * (1.0 + 2.0 ** -6)


@pytest.mark.parametrize("part,K,rows", [(1, 36, 64), (1, 68, 37), (2, 36, 64), (2, 68, 37), (2, 100, 64), (2, 132, 48)])
@pytest.mark.parametrize("what", ["tiny", "huge", "sum", "inf", "nan", "zero", "weight", "weight_sum"])
def test_grouped_ffn_fp32_split_tiles_with_values_out_of_range(what, part, K, rows):
    # one row of an operand beyond what bf16 pieces represent, or sums beyond their range: its tile takes the fp32
    # instruction, bit for bit what 32-row launches give; small rows and rows of zeros stay on the split path.
    # Odd and even numbers of K stages, through the fp32 instruction's two and three LDS stages.
    N, hot = 64 * 321 + 4, rows - 3
    gen = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randn((rows, K), device="cuda", generator=gen)
    b, gate = (torch.randn((N, K), device="cuda", generator=gen) for _ in range(2))

    def run(a):
        T = a.shape[0]
        off = torch.tensor([0, T], dtype=torch.int32, device="cuda")
        out = torch.zeros((T, N), device="cuda")
        if part == 1:
            B.moe_grouped_ffn_part(B.make_shape(T, K, 1, 1, N, si.F32, 1), a, off, gate[None], b[None],
                                   torch.zeros((1, K, N), device="cuda"), out, torch.zeros((T, K), device="cuda"), 1)
        else:
            up = torch.zeros((1, K, N), device="cuda")
            B.moe_grouped_ffn_part(B.make_shape(T, N, 1, 1, K, si.F32, 1), torch.zeros((T, N), device="cuda"), off, up, up,
                                   b[None], a, out, 2)
        torch.cuda.synchronize()
        return out

    ref = run(a)
    if what == "weight":
        b[130] *= 2.0 ** 110                          # third tile of 64 columns: an infinite piece
    elif what == "weight_sum":
        b[130] *= 2.0 ** 85                           # pieces finite, their sums are not
    else:
        a[hot] *= {"tiny": 2.0 ** -50, "huge": 2.0 ** 110, "sum": 2.0 ** 85, "zero": 0.0}.get(what, 1.0)
        if what in ("inf", "nan"):
            a[hot, 5] = float(what)
    got = run(a)
    exact = torch.cat([run(a[:32].clone()), run(a[32:].clone())])
    same = lambda p, q: torch.equal(p.view(torch.int32), q.view(torch.int32))
    if what in ("huge", "sum", "inf", "nan"):
        assert same(got, exact)
    elif what in ("weight", "weight_sum"):
        assert same(got[:, 128:192], exact[:, 128:192])
        assert same(got[:, :128], ref[:, :128]) and same(got[:, 192:], ref[:, 192:])
    else:
        keep = [i for i in range(rows) if i != hot]
        assert same(got[keep], ref[keep]) and not same(got[keep], exact[keep])
        if what == "zero":
            assert bool((got[hot] == 0).all())
    fine = torch.isfinite(exact)
    assert bool((torch.isfinite(got) == fine).all())
    # (by rows and by columns, one of which holds the scaled values)
    exact = exact.where(fine, torch.zeros_like(exact)).double()
    scale = torch.minimum(exact.abs().amax(dim=1, keepdim=True), exact.abs().amax(dim=0, keepdim=True).expand_as(exact))
    if what == "tiny":                                # (a sum of its own size, in a column of ordinary ones)
        scale = exact.abs().amax(dim=1, keepdim=True)
    assert bool(((got.where(fine, torch.zeros_like(got)).double() - exact).abs() <= 8.0 * K ** 0.5 * 2.0 ** -24 * scale).all())


@pytest.mark.parametrize("part", [1, 2])
@pytest.mark.parametrize("E,rows,panels,pieces", [(1, 35, 321, False), (1, 36, 321, True), (1, 64, 320, False), (1, 64, 321, True),
                                                  (3, 36, 161, True), (3, 36, 160, False), (9, 36, 54, True)])
def test_grouped_ffn_fp32_on_both_sides_of_the_split_rule(part, E, rows, panels, pieces):
    # 36 rows per expert and more than 5/4 tiles (64-row tiles of all rows x panels of 64 columns) per CU: pieces, else the fp32
    # instruction.  Which of the two it was shows in the error: the fp32 instruction does not round to nearest and adds four
    # products at a time, 65 times at K = 260 (2.9e-7 of the 2-norm, gated 4.4e-7), the pieces 32, 9 times (up to 1.7e-7).
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 compute units")
    K, N, T = 260, 64 * panels, E * rows
    gen = torch.Generator(device="cuda").manual_seed(E + rows)
    a = torch.randn((T, K), device="cuda", generator=gen)
    b, gate = (torch.randn((E, N, K), device="cuda", generator=gen) * K ** -0.5 for _ in range(2))
    off = torch.arange(E + 1, dtype=torch.int32, device="cuda") * rows
    out = torch.zeros((T, N), device="cuda")
    if part == 1:
        B.moe_grouped_ffn_part(B.make_shape(T, K, E, 1, N, si.F32, 1), a, off, gate, b, torch.zeros((E, K, N), device="cuda"),
                               out, torch.zeros((T, K), device="cuda"), 1)
    else:
        up = torch.zeros((E, K, N), device="cuda")
        B.moe_grouped_ffn_part(B.make_shape(T, N, E, 1, K, si.F32, 1), torch.zeros((T, N), device="cuda"), off, up, up, b, a, out, 2)
    torch.cuda.synchronize()
    rows64 = [a[e * rows:(e + 1) * rows].double() for e in range(E)]
    ref = torch.cat([r @ b[e].double().t().contiguous() for e, r in enumerate(rows64)])
    if part == 1:
        g = torch.cat([r @ gate[e].double().t().contiguous() for e, r in enumerate(rows64)])
        ref = ref * g / (1.0 + torch.exp(-g))
    err = float((out.double() - ref).norm() / ref.norm())
    assert err <= 1e-6 and (err <= 2.2e-7) == pieces, err


@pytest.mark.parametrize("E,T,k", [(8, 330, 2), (5, 650, 1)])
def test_grouped_ffn_fp32_split_tiles_through_the_maps(E, T, k):
    # split tiles of many K stages that read x by src_assign and, with one expert per token, store scaled rows of y
    cfg = si.small_config("f32_split_maps", T=T, d=2052, E=E, k=k, F=2076, dtype=si.F32, renorm=0, seed=E)
    L = si.make_layer(cfg)
    idx = np.stack([np.random.default_rng(t).permutation(E)[:k] for t in range(T)]).astype(np.int32)
    counts, offsets = orc.expert_load(idx, E)
    assert counts.min() > 32
    dst, src = (np.asarray(m, dtype=np.int32) for m in orc.permutation(idx, E))
    args = [dev(offsets)] + [dev(L[n]) for n in ("w1", "w3", "w2")]
    x, src = dev(L["x"]), dev(src)
    new = lambda n: torch.zeros((T * k, n), device="cuda")
    h, yp, hg, yg = new(cfg.F), new(cfg.d), new(cfg.F), new(cfg.d)
    B.moe_grouped_ffn(shape_of(cfg), dev(orc.permute_rows(L["x"], dst, k)), *args, h, yp)
    B.moe_grouped_ffn_gather(shape_of(cfg), x, src, *args, hg, yg)
    torch.cuda.synchronize()
    assert torch.equal(h, hg) and torch.equal(yp, yg)
    if k == 1:
        w = torch.rand(T, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)) + 0.5
        hk, y = new(cfg.F), new(cfg.d)
        B.moe_grouped_ffn_combine_k1(shape_of(cfg), x, src, *args, w, hk, y)
        torch.cuda.synchronize()
        want = torch.empty_like(y)
        want[src.long()] = yp * w[src.long(), None]
        assert torch.equal(h, hk) and torch.equal(y, want)


@pytest.mark.parametrize("dtype,T,d,F,form", [
    (si.F32, 64, 4, 2 ** 23 + 4, "perm"), (si.F32, 64, 4, 2 ** 23 + 4, "k1"),   # 64 activation rows of the down-projection
    (si.F32, 2, 2 ** 23 + 4, 64, "perm"),                                       # 64 weight rows of the up-projection
    (si.BF16, 320, 8, 3355448, "perm"),                                         # 320 activation rows
    (si.BF16, 3, 256, 2 ** 22 + 8, "perm"), (si.BF16, 3, 256, 2 ** 22, "gather"),   # 256 weight rows
    (si.F32, 64, 4, 2 ** 23 - 4, "perm"), (si.BF16, 320, 8, 3355440, "perm")])  # the widest that 32 bits reach
def test_grouped_ffn_rows_around_the_limit_of_32_bit_offsets(dtype, T, d, F, form):
    """One tile's rows of an operand span 2 GiB or more, or just less.  Reference: fp64 sums over slices, on
    the GPU."""
    tdt = torch.float32 if dtype == si.F32 else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(7)

    def randn(shape, std):
        t = torch.empty(shape, dtype=tdt, device="cuda")
        return t.normal_(0.0, std, generator=gen)

    x, w1, w3 = randn((T, d), 1.0), randn((1, F, d), d ** -0.5), randn((1, F, d), d ** -0.5)
    w2 = randn((1, d, F), F ** -0.5)
    src = torch.randperm(T, device="cuda", generator=gen).to(torch.int32) if form != "perm" else None
    scale = torch.rand(T, device="cuda", generator=gen) + 0.5 if form == "k1" else None
    off = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    h, y = torch.zeros((T, F), dtype=tdt, device="cuda"), torch.zeros((T, d), dtype=tdt, device="cuda")
    sh = B.make_shape(T, d, 1, 1, F, dtype, 1)
    if form == "k1":
        B.moe_grouped_ffn_combine_k1(sh, x, src, off, w1, w3, w2, scale, h, y)
    elif form == "gather":
        B.moe_grouped_ffn_gather(sh, x, src, off, w1, w3, w2, h, y)
    else:
        B.moe_grouped_ffn(sh, x, off, w1, w3, w2, h, y)
    torch.cuda.synchronize()
    rows = x if src is None else x[src.long()]

    def product(a, w):                            # a [T, K] times w [N, K] transposed, fp64, sliced along both
        n_step, k_step = max(1, 2 ** 24 // min(w.shape[1], 2 ** 16)), 2 ** 16
        out = torch.zeros((a.shape[0], w.shape[0]), dtype=torch.float64, device="cuda")
        for n in range(0, w.shape[0], n_step):
            for k in range(0, w.shape[1], k_step):
                out[:, n:n + n_step] += a[:, k:k + k_step].double() @ w[n:n + n_step, k:k + k_step].double().t().contiguous()
        return out

    # an fp32 sum of K terms one after the other (rounding 2^-24 of partial sums that grow as a random walk:
    # below sqrt(K) 2^-24 of the result's scale), and a rounding to bf16 where stored so; zeros in
    # place of one row would be off by the whole scale
    def bound(K):
        return 4.0 * K ** 0.5 * 2.0 ** -24 + (2.0 ** -8 if dtype == si.BF16 else 2.0 ** -22)

    g, u = product(rows, w1[0]), product(rows, w3[0])
    ref = g / (1.0 + torch.exp(-g)) * u
    assert float((h.double() - ref).abs().max() / ref.abs().max()) <= bound(d)
    del g, u, ref
    ref = product(h, w2[0])
    if form == "k1":
        scattered = torch.empty_like(ref)
        scattered[src.long()] = ref
        ref = scattered * scale.double()[:, None]
    assert float((y.double() - ref).abs().max() / ref.abs().max()) <= bound(F)


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 47, 64, 65, 130, 255, 257, 319, 320, 321, 336, 641, 1000])
def test_grouped_ffn_even_tiles_every_wave_share(rows):
    # one expert with `rows` rows among others of 600 or 150: its tiles give the waves every count of
    # sub-tiles from 0 to 5, tiles below and at the 320-row limit, and segments that need two or three
    # tiles; mean rows per expert above and below the 384 from which experts of several tiles may keep two
    # weight buffers in the up-projection (d = 128 is a power of two)
    for E, others in ((3, 600), (9, 150)):
        cfg = si.small_config(T=rows + (E - 1) * others, d=128, E=E, k=1, F=256, seed=rows + E)
        L = si.make_layer(cfg)
        idx = np.zeros((cfg.T, 1), dtype=np.int32)
        idx[:rows] = 1
        pos = rows
        for e in range(E):
            if e != 1:
                idx[pos:pos + others] = e
                pos += others
        check_ffn(cfg, L, idx)


@pytest.mark.parametrize("d", [64, 128, 192, 256, 320, 448, 520, 704])
@pytest.mark.parametrize("E,rows,F", [(3, 50, 200), (4, 64, 640), (20, 33, 640), (20, 100, 640), (5, 128, 328), (6, 129, 192)])
def test_grouped_ffn_pieces_of_low_tiles(E, rows, F, d):
    # low tiles of an under-filled round: quarters (E = 3, 4) and halves (E = 20, 81 to 128 tiles) of the
    # weight rows, pieces past the end of the matrix, on either side of the 64- and 128-row limits; whole
    # (the second form gpu_ffn runs) they take the ring and the three and four weight buffers.  1 to 11
    # stages, below and above every ring's depth; widths with K and N tails.
    cfg = si.small_config(T=E * rows, d=d, E=E, k=1, F=F, seed=d + F + rows)
    check_ffn(cfg, si.make_layer(cfg), np.repeat(np.arange(E, dtype=np.int32), rows)[:, None])


ROUND_CASES = [
    # (rows per expert, d, F): enough tiles for whole rounds of the chip's 256 compute units plus a
    # last round that is under-filled (its tiles are cut along their rows), just over half full
    # (left whole) or absent; every element of h and y_perm is compared
    ([2048] * 8, 128, 640),                      # up 280 tiles (1 round + 24), down 56 (a fifth of a round)
    ([1500] * 16, 512, 384),                     # up 240 (under a round, whole tiles), down 160
    ([3000, 17, 0, 2500, 64, 700, 1, 4000, 0, 333, 2100, 65, 1290, 1280, 320, 321], 256, 1152),
    ([1024] * 9, 1024, 512),                     # up 144, down 144: just over half a round, not cut
    ([640] * 40, 128, 896),                      # up 560 (2 rounds + 48), down 80
]


@pytest.mark.parametrize("rows,d,F", ROUND_CASES, ids=lambda v: str(v) if isinstance(v, int) else f"E{len(v)}")
def test_grouped_ffn_whole_rounds_and_under_filled_last_rounds(rows, d, F):
    cfg = si.small_config(T=sum(rows), d=d, E=len(rows), k=1, F=F, seed=len(rows) + d + F)
    L = si.make_layer(cfg)
    idx = np.repeat(np.arange(len(rows), dtype=np.int32), rows).reshape(-1, 1)
    check_ffn(cfg, L, idx)


@pytest.mark.parametrize("d", [192, 256, 520])
@pytest.mark.parametrize("rows", [(544, 540, 530, 560), (272, 80, 80, 80, 80, 80, 80), (130, 40, 40, 40), (300, 257, 400, 640)])
def test_grouped_ffn_tiles_of_one_expert_on_both_sides_of_a_pipeline_s_limit(rows, d):
    # experts of two tiles with one up to and one above 256 rows, which both take the higher one's pipeline,
    # and with one up to and one above 128 or 64, which take their own; the first and last case have the
    # mean rows at which a power-of-two reduction (d = 256) keeps two weight buffers in the up-projection
    cfg = si.small_config(T=sum(rows), d=d, E=len(rows), k=1, F=384 if d != 520 else 392, seed=d + rows[0])
    check_ffn(cfg, si.make_layer(cfg), np.repeat(np.arange(len(rows), dtype=np.int32), rows)[:, None])


SPLIT_CASES = [
    # (shape, whether some tile must have been split); a GEMM is eligible from K = 6144 on
    (dict(T=600, d=1024, E=2, k=1, F=6144), True),    # even tiles, down-projection cut in 4
    (dict(T=64, d=1024, E=4, k=2, F=6144), True),     # ring tiles (32 rows per expert)
    (dict(T=600, d=6144, E=2, k=1, F=256), True),     # up-projection (gated) cut in 4
    (dict(T=700, d=1024, E=2, k=1, F=6144, seed=11), None),   # 350 rows per expert: two even tiles of 176 rows each
    (dict(T=300, d=1024, E=2, k=1, F=2048), False),   # reductions too short: exactly the plain call
    # given rows per expert: four weight buffers (65 to 128 rows), both GEMMs
    (dict(rows=(80, 66, 100, 125), d=1024, F=6144), True),
    (dict(rows=(80, 66, 100, 128), d=6144, F=256), True),
    (dict(rows=(200, 130, 256), d=6144, F=256), True),       # three, gated
    (dict(rows=(544, 560), d=1024, F=6144), True),           # tiles of one expert on both sides of 256 rows
    (dict(rows=(400, 410), d=8192, F=256), True),            # gated, two buffers for experts of two tiles
    (dict(rows=(700, 690), d=1024, F=6144), True),           # 640 rows and more: the default policy's kernels
    (dict(rows=(700, 690), d=6144, F=256), True),
    (dict(rows=(500, 40, 40, 40, 30, 1, 65, 190), d=1024, F=6144), True),   # a hot expert in tiles of up to 192 rows
]


@pytest.mark.parametrize("case,expect_split", SPLIT_CASES,
                         ids=lambda c: "_".join(f"{n}{v}" for n, v in c.items()) if isinstance(c, dict) else "")
@pytest.mark.parametrize("gathered", [False, True])
def test_grouped_ffn_with_split_tiles(case, expect_split, gathered):
    """moe_grouped_ffn_ws: tiles of an under-filled last round are computed in parts along K and
    added up by the launch after the GEMM.  Oracle parity, run-to-run identical bits whatever the
    workspace held before, rows within a bf16 step of the call without a workspace; where the
    case says so, the split did happen (some bits differ) or cannot (identical bits)."""
    case = dict(case)
    rows = case.pop("rows", None)
    if rows:
        case.update(T=sum(rows), E=len(rows), k=1)
    cfg = si.small_config(**case)
    L = si.make_layer(cfg)
    if rows:
        idx = np.random.default_rng(len(rows)).permutation(np.repeat(np.arange(cfg.E, dtype=np.int32), rows))[:, None]
    else:
        idx, _, _ = orc.route(L["x"], L["w_gate"], cfg.k, cfg.renorm)
    _, offsets = orc.expert_load(idx, cfg.E)
    dst, src = orc.permutation(idx, cfg.E)
    x_perm = orc.permute_rows(L["x"], dst, cfg.k)
    ry, rh = orc.grouped_ffn(x_perm, offsets, L["w1"], L["w3"], L["w2"], return_h=True)
    sh = shape_of(cfg)
    A = cfg.T * cfg.k
    nb = B.moe_ffn_workspace_bytes(sh)
    d_x = dev(L["x"]) if gathered else dev(x_perm)
    d_src = dev(src) if gathered else None
    d_off, w1, w3, w2 = dev(offsets), dev(L["w1"]), dev(L["w3"]), dev(L["w2"])
    outs = []
    for fill in (0, 0x7F):                           # 0x7F7F7F7F is a large finite float: stale data would show
        ws = torch.full((nb,), fill, dtype=torch.uint8, device="cuda")
        h = torch.zeros((A, cfg.F), dtype=tdtype(cfg), device="cuda")
        yp = torch.zeros((A, cfg.d), dtype=tdtype(cfg), device="cuda")
        B.moe_grouped_ffn_ws(sh, d_x, d_src, d_off, w1, w3, w2, h, yp, 3, ws, nb)
        torch.cuda.synchronize()
        outs.append((h, yp))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    h, yp = outs[0]
    tol = tol_of(cfg.dtype)
    assert rel_err(orc.to_f64(host(h)), rh) <= tol
    assert rel_err(orc.to_f64(host(yp)), ry) <= tol
    # against the call without a workspace: the same rows up to the grouping of the fp32 sum
    h0 = torch.zeros_like(h)
    y0 = torch.zeros_like(yp)
    B.moe_grouped_ffn_ws(sh, d_x, d_src, d_off, w1, w3, w2, h0, y0, 3, None, 0)
    torch.cuda.synchronize()
    assert (h.float() - h0.float()).abs().max().item() <= 2.0 ** -7 * h0.float().abs().max().item()
    assert (yp.float() - y0.float()).abs().max().item() <= 2.0 ** -6 * y0.float().abs().max().item()
    same = torch.equal(h, h0) and torch.equal(yp, y0)
    if expect_split is True:
        assert not same, "no tile was split"
    elif expect_split is False:
        assert same


def test_grouped_ffn_skewed_and_empty_experts():
    cfg = si.small_config(T=700, d=128, E=8, k=2, F=256)
    L = si.make_layer(cfg)
    idx = np.zeros((cfg.T, 2), dtype=np.int32)
    idx[:, 0] = 2                                     # 700 rows: 256-row tiles with a tail
    idx[:, 1] = np.where(np.arange(cfg.T) < 5, 6, 4)  # 5 rows and 695 rows; 5 experts empty
    check_ffn(cfg, L, idx)


def test_identity_experts_reproduce_the_input_on_gpu():
    # closed form: W1 rows = c*e0, W3 = [I;0], W2 = [I/silu(c), 0]  =>  E(x) = x when x[:,0] = 1
    T, d, E, k, F = 200, 128, 4, 2, 192
    cfg = si.small_config(T=T, d=d, E=E, k=k, F=F, dtype=si.F32)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    x = L["x"].copy()
    x[:, 0] = 1.0
    c = 1.5
    s0 = c / (1.0 + np.exp(-c))
    w1 = np.zeros((E, F, d), np.float32); w1[:, :, 0] = c
    w3 = np.zeros((E, F, d), np.float32); w3[:, :d, :d] = np.eye(d)
    w2 = np.zeros((E, d, F), np.float32); w2[:, :d, :d] = np.eye(d) / s0
    buf = layer.MoeBuffers(T, d, E, k, F, cfg.dtype, 1)
    buf.forward(dev(x), dev(L["w_gate"]), dev(w1), dev(w3), dev(w2))
    torch.cuda.synchronize()
    assert rel_err(host(buf.y), x) <= 1e-5


# ----------------------------------------------------------------------------- combine
@pytest.mark.parametrize("case", [dict(T=300, d=256, E=8, k=2), dict(T=257, d=1032, E=64, k=6),
                                  dict(T=31, d=4096, E=128, k=8),
                                  dict(T=40, d=100, E=6, k=3, dtype=si.F32)],
                         ids=lambda c: "T{T}_d{d}_k{k}".format(**c))
def test_combine_matches_oracle(case):
    cfg = si.small_config(F=64, **case)
    L = si.make_layer(cfg, parts=("x", "w_gate"))
    idx, w, _ = orc.route(L["x"], L["w_gate"], cfg.k, cfg.renorm)
    dst, _ = orc.permutation(idx, cfg.E)
    # any rows will do as "expert outputs": draw them with the generator
    yp = si.make_layer(si.small_config(T=cfg.A, d=cfg.d, E=1, k=1, F=8, dtype=cfg.dtype, seed=99),
                       parts=("x",))["x"]
    y = torch.zeros((cfg.T, cfg.d), dtype=tdtype(cfg), device="cuda")
    B.moe_combine(shape_of(cfg), dev(yp), dev(dst), dev(w), y)
    torch.cuda.synchronize()
    ref = orc.combine(yp, dst, w)
    assert rel_err(orc.to_f64(host(y)), ref) <= (1e-6 if cfg.dtype == si.F32 else 4e-3)


@pytest.mark.parametrize("T,d,k,dtype", [(1, 1016, 1, si.BF16), (5, 1024, 5, si.BF16), (3, 1032, 2, si.BF16),
                                         (4, 2048, 4, si.BF16), (6, 2056, 3, si.BF16), (7, 508, 1, si.F32),
                                         (2, 512, 5, si.F32), (9, 516, 2, si.F32)])
def test_combine_at_the_edges_of_its_column_slabs(T, d, k, dtype):
    """A wave sums 2 KiB of a row: rows one chunk short of, equal to and one chunk past whole slabs, and
    tokens that do not fill a block of four."""
    cfg = si.small_config(T=T, d=d, E=8, k=k, F=64, dtype=dtype)
    rng = np.random.default_rng(d)
    w = rng.random((T, k), dtype=np.float32)
    dst = rng.permutation(T * k).astype(np.int32)
    yp = si.make_layer(si.small_config(T=T * k, d=d, E=1, k=1, F=8, dtype=dtype, seed=99), parts=("x",))["x"]
    y = torch.zeros((T, d), dtype=tdtype(cfg), device="cuda")
    B.moe_combine(shape_of(cfg), dev(yp), dev(dst), dev(w), y)
    torch.cuda.synchronize()
    # the same bounds as above: k fp32 products and sums, for bf16 one rounding to 8 bits
    assert rel_err(orc.to_f64(host(y)), orc.combine(yp, dst, w)) <= (1e-6 if dtype == si.F32 else 4e-3)


@pytest.mark.parametrize("chunks", [192, 193, 384, 385, 512, 513, 640, 641, 769, 896, 897, 960, 961, 1025])
@pytest.mark.parametrize("dtype", [si.BF16, si.F32])
def test_combine_in_slabs_of_2_3_and_4_kib(chunks, dtype):
    # rows of so many 16-byte chunks take waves of 2, 3 or 4 KiB, whichever gives an odd number of slabs
    T, k = 5, 3
    cfg = si.small_config(T=T, d=chunks * (8 if dtype == si.BF16 else 4), E=8, k=k, F=64, dtype=dtype)
    rng = np.random.default_rng(chunks)
    w = rng.random((T, k), dtype=np.float32)
    dst = rng.permutation(T * k).astype(np.int32)
    yp = si.make_layer(si.small_config(T=T * k, d=cfg.d, E=1, k=1, F=8, dtype=dtype, seed=99), parts=("x",))["x"]
    y = torch.zeros((T, cfg.d), dtype=tdtype(cfg), device="cuda")
    B.moe_combine(shape_of(cfg), dev(yp), dev(dst), dev(w), y)
    torch.cuda.synchronize()
    # k fp32 products and sums, for bf16 one rounding to 8 bits
    assert rel_err(orc.to_f64(host(y)), orc.combine(yp, dst, w)) <= (1e-6 if dtype == si.F32 else 4e-3)


# ----------------------------------------------------------------------------- whole layer
LAYER_CASES = [
    si.CONFIGS["tiny"],
    si.small_config("bf16_small", T=300, d=256, E=8, k=2, F=384),
    si.small_config("bf16_fine", T=500, d=256, E=64, k=6, F=128, renorm=0),
    si.small_config("bf16_big_tiles", T=1400, d=128, E=2, k=2, F=256),
    si.small_config("bf16_decode_like", T=32, d=512, E=128, k=8, F=192),
    si.small_config("bf16_skew", T=600, d=256, E=64, k=6, F=128, renorm=0, zipf_alpha=1.2,
                    zipf_scale=0.9, empty_tail=4),
    si.small_config("bf16_limits", T=100, d=128, E=256, k=64, F=64),       # the largest E and k
    si.small_config("bf16_top1", T=700, d=128, E=16, k=1, F=192),          # one expert per token
    si.small_config("bf16_all_experts", T=150, d=128, E=8, k=8, F=64, renorm=0),   # k = E
    si.small_config("bf16_many_tokens", T=20000, d=64, E=8, k=2, F=64),    # many dispatch blocks
    si.small_config("f32_odd", T=130, d=100, E=12, k=3, F=52, dtype=si.F32),
]


@pytest.mark.parametrize("cfg", LAYER_CASES, ids=lambda c: c.name)
def test_layer_end_to_end(cfg):
    L = si.make_layer(cfg)
    ref = orc.moe_layer(L["x"], L["w_gate"], L["w1"], L["w3"], L["w2"], cfg.k, cfg.renorm,
                        L["gate_bias"])
    buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
    args = [dev(L[n]) for n in ("x", "w_gate", "w1", "w3", "w2")]
    buf.forward(*args, gate_bias=dev(L["gate_bias"]), export_scores=True)
    torch.cuda.synchronize()
    first = {n: host(getattr(buf, n)).copy() for n in
             ("topk_idx", "topk_w", "counts", "offsets", "dst_row", "src_assign", "x_perm", "h",
              "y_perm", "y")}
    for n in ("topk_idx", "counts", "offsets", "dst_row", "src_assign", "x_perm"):
        assert np.array_equal(first[n], ref[n]), n
    assert np.all(np.abs(first["topk_w"] - ref["topk_w"]) <= 1e-5 * ref["topk_w"] + 1e-9)
    tol = tol_of(cfg.dtype)
    for n in ("h", "y_perm", "y"):
        e = rel_err(orc.to_f64(first[n]), ref[n])
        assert e <= tol, f"{n}: {e:.3e}"
    assert first["counts"].sum() == cfg.A
    # determinism: a second run gives the same bits everywhere
    buf.forward(*args, gate_bias=dev(L["gate_bias"]), export_scores=True)
    torch.cuda.synchronize()
    for n, v in first.items():
        assert np.array_equal(host(getattr(buf, n)), v), f"{n} differs between two runs"


def test_layer_replays_from_a_hip_graph():
    """The four calls captured into one HIP graph replay to the eager bits.  Eager work and
    synchronisations sit between the replays; no call allocates or clears memory."""
    cfg = si.small_config("bf16_graph", T=1400, d=128, E=2, k=2, F=256)
    L = si.make_layer(cfg)
    buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
    args = [dev(L[n]) for n in ("x", "w_gate", "w1", "w3", "w2")]
    bias = dev(L["gate_bias"])
    names = ("topk_idx", "topk_w", "counts", "offsets", "dst_row", "src_assign", "x_perm", "h",
             "y_perm", "y")
    buf.forward(*args, gate_bias=bias)
    torch.cuda.synchronize()
    eager = {n: host(getattr(buf, n)).copy() for n in names}
    ref = orc.moe_layer(L["x"], L["w_gate"], L["w1"], L["w3"], L["w2"], cfg.k, cfg.renorm,
                        L["gate_bias"])
    assert rel_err(orc.to_f64(eager["y"]), ref["y"]) <= tol_of(cfg.dtype)

    graph = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        buf.forward(*args, gate_bias=bias)          # first use of this stream happens outside the capture
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        buf.forward(*args, gate_bias=bias)
    torch.cuda.synchronize()
    for rep in range(3):
        for n in names:                             # eager fills between the replays
            getattr(buf, n).zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n in names:
            assert np.array_equal(host(getattr(buf, n)), eager[n]), f"replay {rep}: {n} differs"


def test_layer_with_split_tiles_replays_from_a_hip_graph():
    """The layer with the split-tile workspace (the down-projection's tiles cut along K, summed by
    the launch after the GEMM) captured into a HIP graph: every replay gives the eager bits, with
    the workspace overwritten between the replays."""
    cfg = si.small_config("bf16_graph_split", T=64, d=256, E=4, k=2, F=6144)
    L = si.make_layer(cfg)
    buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm, split_tiles=True)
    plain = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
    args = [dev(L[n]) for n in ("x", "w_gate", "w1", "w3", "w2")]
    names = ("topk_idx", "counts", "dst_row", "h", "y_perm", "y")
    buf.forward(*args)
    plain.forward(*args)
    torch.cuda.synchronize()
    eager = {n: host(getattr(buf, n)).copy() for n in names}
    ref = orc.moe_layer(L["x"], L["w_gate"], L["w1"], L["w3"], L["w2"], cfg.k, cfg.renorm, None)
    assert rel_err(orc.to_f64(eager["y"]), ref["y"]) <= tol_of(cfg.dtype)
    assert not np.array_equal(eager["y_perm"], host(plain.y_perm)), "no tile was split"
    graph = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        buf.forward(*args)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=s):
        buf.forward(*args)
    torch.cuda.synchronize()
    for rep in range(3):
        for n in names:
            getattr(buf, n).zero_()
        buf.ffn_ws.fill_(0x7F)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n in names:
            assert np.array_equal(host(getattr(buf, n)), eager[n]), f"replay {rep}: {n} differs"


@pytest.mark.parametrize("cfg", LAYER_CASES, ids=lambda c: c.name)
def test_ffn_reading_x_through_the_permutation_gives_the_same_bits(cfg):
    """moe_grouped_ffn_gather (no x_perm) against moe_grouped_ffn on the materialised x_perm."""
    L = si.make_layer(cfg)
    buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
    args = [dev(L[n]) for n in ("x", "w_gate", "w1", "w3", "w2")]
    bias = dev(L["gate_bias"])
    buf.forward(*args, gate_bias=bias)
    torch.cuda.synchronize()
    want = {n: host(getattr(buf, n)).copy() for n in ("src_assign", "h", "y_perm", "y")}
    for n in ("x_perm", "h", "y_perm", "y"):
        getattr(buf, n).zero_()
    buf.forward(*args, gate_bias=bias, gather_in_ffn=True)
    torch.cuda.synchronize()
    for n, v in want.items():
        assert np.array_equal(host(getattr(buf, n)), v), n
    assert not host(buf.x_perm).any()                   # x_perm was not touched
    ref = orc.moe_layer(L["x"], L["w_gate"], L["w1"], L["w3"], L["w2"], cfg.k, cfg.renorm,
                        L["gate_bias"])
    assert rel_err(orc.to_f64(host(buf.y)), ref["y"]) <= tol_of(cfg.dtype)


def test_ffn_gather_rejects_missing_map_and_survives_bad_entries():
    cfg = si.small_config("gather_bad", T=200, d=128, E=4, k=2, F=128)
    L = si.make_layer(cfg)
    buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
    args = [dev(L[n]) for n in ("x", "w_gate", "w1", "w3", "w2")]
    buf.forward(*args, gather_in_ffn=True)
    with pytest.raises(B.MoeError):
        B.moe_grouped_ffn_gather(buf.shape, args[0], None, buf.offsets, args[2], args[3], args[4],
                                 buf.h, buf.y_perm)
    # entries outside [0, T*k) are clamped to a valid row: values unspecified, no fault
    bad = buf.src_assign.clone()
    bad[::7] = 1 << 30
    bad[3::11] = -5
    B.moe_grouped_ffn_gather(buf.shape, args[0], bad, buf.offsets, args[2], args[3], args[4], buf.h,
                             buf.y_perm)
    torch.cuda.synchronize()
    assert np.isfinite(orc.to_f64(host(buf.y_perm))).all()


def test_two_host_threads_on_two_streams():
    """The header promises that calls from several host threads are independent (the library keeps
    no state of its own).  Two threads, each with its own stream and buffers, run the layer
    repeatedly at the same time; every result equals the one obtained alone."""
    import threading
    cfgs = [si.small_config("thr_a", T=1400, d=128, E=2, k=2, F=256),
            si.small_config("thr_b", T=900, d=256, E=4, k=2, F=128, seed=11)]
    jobs = []
    for cfg in cfgs:
        L = si.make_layer(cfg)
        args = [dev(L[n]) for n in ("x", "w_gate", "w1", "w3", "w2")]
        buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
        buf.forward(*args)
        torch.cuda.synchronize()
        jobs.append((cfg, args, buf, host(buf.y).copy(), torch.cuda.Stream()))
    errors = []

    def run(job):
        cfg, args, buf, want, stream = job
        try:
            for it in range(20):
                with torch.cuda.stream(stream):
                    buf.y.zero_()
                    buf.forward(*args, stream=stream, gather_in_ffn=bool(it & 1))
                stream.synchronize()
                if not np.array_equal(host(buf.y), want):
                    errors.append(f"{cfg.name}: iteration {it} differs")
                    return
        except Exception as exc:  # noqa: BLE001
            errors.append(f"{cfg.name}: {exc!r}")

    threads = [threading.Thread(target=run, args=(j,)) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
    assert not any(t.is_alive() for t in threads), "a thread did not finish"
    assert not errors, errors


# ----------------------------------------------------------------------------- k = 1: combine in the FFN
@pytest.mark.parametrize("cfg", [
    si.small_config("k1_even", T=1500, d=256, E=3, k=1, F=384, renorm=0),       # even tiles, several per expert
    si.small_config("k1_ring", T=300, d=128, E=8, k=1, F=256, renorm=0, seed=5),  # ring tiles
    si.small_config("k1_odd", T=200, d=96, E=4, k=1, F=160, renorm=0, seed=6),  # bf16, no MFMA shape
    si.small_config("k1_f32", T=150, d=64, E=4, k=1, F=96, dtype=si.F32, renorm=0, seed=7),
], ids=lambda c: c.name)
def test_ffn_with_the_combine_folded_in_for_one_expert_per_token(cfg):
    """moe_grouped_ffn_combine_k1 against the oracle's layer and against the two-call form (which
    rounds y_perm before the weight is applied: at most one more rounding)."""
    L = si.make_layer(cfg)
    ref = orc.moe_layer(L["x"], L["w_gate"], L["w1"], L["w3"], L["w2"], cfg.k, cfg.renorm, L["gate_bias"])
    args = [dev(L[n]) for n in ("x", "w_gate", "w1", "w3", "w2")]
    buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
    buf.forward(*args, gather_in_ffn=True)
    torch.cuda.synchronize()
    two_calls = orc.to_f64(host(buf.y))
    h_two = host(buf.h).copy()
    buf.y.zero_()
    buf.y_perm.fill_(7)                              # must stay untouched
    buf.forward(*args, combine_in_ffn=True)
    torch.cuda.synchronize()
    fused = orc.to_f64(host(buf.y))
    assert np.array_equal(host(buf.topk_idx), ref["topk_idx"])
    assert np.array_equal(host(buf.h), h_two)
    assert (orc.to_f64(host(buf.y_perm)) == 7).all()
    tol = tol_of(cfg.dtype)
    assert rel_err(fused, ref["y"]) <= tol
    row_scale = np.abs(ref["y"]).max(axis=1) + 1e-30
    assert (np.abs(fused - ref["y"]).max(axis=1) / row_scale).max() <= 4 * tol
    # one rounding of the storage type apart from the two-call form, element by element
    ulp = 2.0 ** -8 if cfg.dtype == si.BF16 else 2.0 ** -23
    assert np.all(np.abs(fused - two_calls) <= 2 * ulp * np.abs(two_calls) + 1e-30)
    # every row of y was written
    assert (np.abs(fused).max(axis=1) > 0).all()


def test_ffn_combine_k1_rejects_layers_with_more_experts_per_token():
    cfg = si.small_config("k2", T=64, d=64, E=4, k=2, F=64)
    buf = layer.MoeBuffers(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, cfg.dtype, cfg.renorm)
    z = torch.zeros((cfg.E, cfg.F, cfg.d), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.MoeError) as err:
        B.moe_grouped_ffn_combine_k1(buf.shape, buf.y, buf.src_assign, buf.offsets, z, z, z, buf.topk_w,
                                     buf.h, buf.y)
    assert err.value.code == -2
