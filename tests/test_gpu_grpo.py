"""Parity of the GRPO advantage / clipped-ratio objective calls with the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import npy, to_dev

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
RTOL = 2e-6        # fp64 arithmetic on both sides; the results are rounded to fp32 once (6e-8) and the
                   # per-rollout weight is passed as fp32 (6e-8); 2e-6 leaves margin for cancellation in J


@pytest.fixture(scope="module")
def A():
    import paper_2603_24840_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def W():
    from paper_2603_24840_amd import workloads
    return workloads


def f32(x):
    return float(np.float32(x))


def dev_i64(a):
    return torch.tensor(np.asarray(a, dtype=np.int64), device=DEV)


@pytest.mark.parametrize("sizes,ddof,eps", [([4] * 64, 0, 0.0), ([8, 1, 0, 3, 64, 65, 200, 2], 0, 0.0),
                                            ([5, 7, 1, 16], 1, 0.0), ([4, 4, 6], 0, 1e-6)])
def test_advantage_matches_oracle(A, sizes, ddof, eps):
    print("[case] grpo_advantage sizes=%s ddof=%d" % (sizes[:8], ddof), flush=True)
    off = np.concatenate([[0], np.cumsum(sizes)])
    N = int(off[-1])
    g = torch.Generator(device=DEV); g.manual_seed(N + ddof)
    reward = (torch.rand(N, generator=g, device=DEV) < 0.4).to(torch.float32)
    reward[:sizes[0]] = 1.0                                  # first group: all equal -> zero advantage
    if len(sizes) > 5:
        reward[off[5]:off[6]] = torch.randn(sizes[5], generator=g, device=DEV)   # real-valued rewards
    adv, wgt = A.arrol_grpo_advantage(reward, dev_i64(off), ddof=ddof, eps=eps)
    torch.cuda.synchronize()
    ref = O.grpo_advantage(npy(reward), off, ddof=ddof, eps=f32(eps))
    assert np.all(np.abs(npy(adv) - ref) <= RTOL * np.abs(ref)), float(np.abs(npy(adv) - ref).max())
    assert np.all(npy(adv)[:sizes[0]] == 0.0)
    for gi, n in enumerate(sizes):
        if n:
            assert np.all(npy(wgt)[off[gi]:off[gi + 1]] == np.float32(1.0 / (n * len(sizes))))


def run_objective(A, lens, sizes, seed, eps_low=0.2, eps_high=0.2, beta=0.0, drift=0.3):
    cu = np.concatenate([[0], np.cumsum(lens)])
    off = np.concatenate([[0], np.cumsum(sizes)])
    assert off[-1] == len(lens)
    T = int(cu[-1])
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    logp_ref = -torch.rand(max(T, 1), generator=g, device=DEV)[:T] * 4
    logp = logp_ref + torch.randn(max(T, 1), generator=g, device=DEV)[:T] * drift
    reward = (torch.rand(len(lens), generator=g, device=DEV) < 0.5).to(torch.float32)
    # advantages: the oracle's, rounded to the interface's fp32, feed both sides; the per-rollout weights
    # 1/(group size * groups) are what arrol_grpo_advantage hands to the objective (checked in the test above)
    adv_o = O.grpo_advantage(npy(reward), off).astype(np.float32)
    adv = to_dev(adv_o, DEV)
    _, wgt = A.arrol_grpo_advantage(reward, dev_i64(off))
    J, grad, n_clip = A.arrol_grpo_objective(logp, logp_ref, dev_i64(cu), adv, wgt, eps_low, eps_high, beta)
    torch.cuda.synchronize()
    Jo, go, co = O.grpo_objective(npy(logp), npy(logp_ref), cu, adv_o, off, f32(eps_low), f32(eps_high), f32(beta))
    scale = max(abs(Jo), float(np.mean(np.abs(adv_o))) if len(lens) else 0.0, 1e-30)
    assert abs(float(J) - Jo) <= RTOL * scale, (float(J), Jo)
    assert int(n_clip) == co
    err = np.abs(npy(grad).astype(np.float64) - go)
    assert np.all(err <= RTOL * np.abs(go) + 1e-30), float(err.max())
    return float(J), co, T


@pytest.mark.parametrize("beta", [0.0, 0.04])
@pytest.mark.parametrize("eps_low,eps_high", [(0.2, 0.2), (0.2, 0.28)])
def test_objective_matches_oracle_ragged(A, eps_low, eps_high, beta):
    print("[case] grpo_objective eps=(%g,%g) beta=%g" % (eps_low, eps_high, beta), flush=True)
    lens = [1, 2, 0, 255, 256, 257, 1000, 3, 64, 700, 5, 9]
    J, n_clip, T = run_objective(A, lens, [4, 2, 6], seed=int(beta * 100) + 7, eps_low=eps_low, eps_high=eps_high,
                                 beta=beta)
    assert 0 < n_clip < T


def test_objective_on_policy_and_degenerate_inputs(A):
    print("[case] grpo_objective on-policy / empty", flush=True)
    run_objective(A, [10, 20, 30, 40], [4], seed=3, drift=0.0)          # ratio 1: nothing clipped
    run_objective(A, [0, 0, 0], [3], seed=4)                            # only empty rollouts
    J, grad, n_clip = A.arrol_grpo_objective(torch.empty(0, device=DEV), torch.empty(0, device=DEV), dev_i64([0]),
                                             torch.empty(0, device=DEV), torch.empty(0, device=DEV))
    torch.cuda.synchronize()
    assert float(J) == 0.0 and int(n_clip) == 0


def test_objective_benchmark_shape(A, W):
    """llama1b survivors: 64 groups of K = 4 rollouts with the benchmark's response-length mix."""
    cfg = W.CONFIGS["llama1b"]
    lens = W.response_lengths(cfg).numpy().tolist()
    print("[case] grpo_objective llama1b n=%d T=%d" % (len(lens), sum(lens)), flush=True)
    run_objective(A, lens, [cfg.K] * (len(lens) // cfg.K), seed=11, beta=0.01)


def test_objective_at_extreme_ratios(A):
    """exp(u) is the reciprocal of exp(-u) where that keeps its bits: log-ratios around the ends of that range (ln 1e300 =
    690.8), beyond the fp64 range, infinite, undefined and zero, both signs of the advantage."""
    print("[case] grpo_objective extreme ratios", flush=True)
    u = np.array([0.0, 1e-7, -1e-7, 1.0, -1.0, 87.0, -87.0, 690.5, 691.0, -690.5, -691.0, 709.5, -709.5, 750.0, -750.0, np.inf, -np.inf, np.nan])
    lens, beta = [len(u)] * 2, 0.5
    ref = np.concatenate([u, u]).astype(np.float32)
    adv, cu = np.array([1.0, -0.5], np.float32), np.array([0, len(u), 2 * len(u)])
    J, grad, n_clip = A.arrol_grpo_objective(torch.zeros(len(ref), device=DEV), to_dev(ref, DEV), dev_i64(cu), to_dev(adv, DEV),
                                             torch.full((2,), 0.5, device=DEV), 0.2, 0.28, beta)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        u64, a = ref.astype(np.float64), np.repeat(adv.astype(np.float64), lens)
        ratio = np.exp(-u64)
        plain, clamped = ratio * a, np.fmin(np.fmax(ratio, 1.0 - f32(0.2)), 1.0 + f32(0.28)) * a
        want = ((np.where(plain <= clamped, plain, 0.0) - beta * (1.0 - np.exp(u64))) * (0.5 / len(u))).astype(np.float32)
        clipped = int(np.sum(clamped < plain))
    got = npy(grad)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    ok = np.isfinite(want)
    # two rounded fp64 terms that cancel near u = 0 (each up to 1), then one rounding to fp32
    assert np.all(np.abs(got[ok] - want[ok]) <= 1e-7 * np.abs(want[ok]) + 1e-15 * 0.5 / len(u) * 4)
    assert np.array_equal(np.signbit(got[~ok & ~np.isnan(want)]), np.signbit(want[~ok & ~np.isnan(want)]))
    assert int(n_clip) == clipped and np.isnan(float(J))


# A rollout goes in steps of four, two and one tokens a thread, by its own length: lengths on both sides of each step's line for workgroups of
# 256 threads and of 512 (a mean above 1,024), none, one, and a rollout of many steps among short ones
@pytest.mark.parametrize("N", [256, 512])
def test_objective_steps_by_rollout_length(A, N):
    print("[case] grpo_objective steps of %d threads" % N, flush=True)
    lens = np.array([0, 1, 63, N - 1, N, N + 1, 2 * N - 1, 2 * N, 2 * N + 1, 3 * N - 1, 3 * N, 3 * N + 1, 4 * N, 4 * N + 1, 5 * N, 5 * N + 1, 6 * N + 1, 7 * N,
                     7 * N + 1, 8 * N + 3, 3, 0] + [20 * N + 7] * (N == 512) + [64] * (20 if N == 256 else 0))
    T, n, beta = int(lens.sum()), len(lens), 0.04
    assert (T // n > 1024) == (N == 512)
    rng = np.random.default_rng(N)
    rng.shuffle(lens)
    logp, ref = ((rng.normal(size=T) * 0.2 - 2).astype(np.float32) for _ in range(2))
    adv, weight = rng.normal(size=n).astype(np.float32), rng.random(n).astype(np.float32)
    ws = torch.empty(16 * n, dtype=torch.uint8, device=DEV)                  # room for one part a rollout
    J, grad, n_clip = A.arrol_grpo_objective(to_dev(logp, DEV), to_dev(ref, DEV), dev_i64(np.concatenate([[0], np.cumsum(lens)])), to_dev(adv, DEV),
                                             to_dev(weight, DEV), 0.2, 0.28, beta, workspace=ws)
    torch.cuda.synchronize()
    u, a = ref.astype(np.float64) - logp.astype(np.float64), np.repeat(adv.astype(np.float64), lens)
    scale = np.repeat(weight.astype(np.float64) / np.maximum(lens, 1), lens)
    ratio, eu = np.exp(-u), np.exp(u)
    plain, clamped = ratio * a, np.clip(ratio, 1.0 - f32(0.2), 1.0 + f32(0.28)) * a
    terms = (np.minimum(plain, clamped) - f32(beta) * (eu - u - 1.0)) * scale
    want = (np.where(plain <= clamped, plain, 0.0) - f32(beta) * (1.0 - eu)) * scale
    assert np.all(np.abs(npy(grad) - want) <= 1e-7 * np.abs(want) + 4e-15 * scale)      # one rounding to fp32; exponentials within 2 ulp
    assert int(n_clip) == int(np.sum(clamped < plain))
    assert abs(float(J) - terms.sum()) <= 4e-15 * np.abs(terms).sum()


# The exponentials themselves: with a clip range that never binds, weight 1 and one token, J is exp(-u) for advantage 1 and beta 0, and
# -(exp(u) - u - 1) for advantage 0 and beta 1, where from u = 60 on u + 1 is less than half an ulp of exp(u).  Rounded are r, sinh r, their
# sum with cosh r - 1 (a quarter of an ulp each where the result is just below a power of two, less elsewhere) and the last
# addition (half a one): 1.25, and for what the polynomials' terms before add 1.3; evenly distributed errors of those sizes have a root mean
# square of 0.38.
def test_objective_exponentials_to_the_last_bit(A):
    rng = np.random.default_rng(3)
    u = np.concatenate([rng.uniform(-690, 690, 300), rng.uniform(-80, 80, 300), rng.normal(size=300) * 0.2]).astype(np.float32)
    one, cu, lp = torch.ones(1, device=DEV), dev_i64(np.array([0, 1])), torch.zeros(1, device=DEV)
    ws, ref = torch.empty(128, dtype=torch.uint8, device=DEV), to_dev(u, DEV)
    down, up = (npy(torch.stack([A.arrol_grpo_objective(lp, ref[i:i + 1], cu, adv, one, 1.0, 3e38, beta, want_grad=False, workspace=ws)[0][0]
                                 for i in range(len(u))])) for adv, beta in ((one, 0.0), (one * 0, 1.0)))
    x = u.astype(np.longdouble)
    for got, want, at in ((down, np.exp(-x), np.abs(u) < 80), (-up, np.exp(x) - x - 1, u > 60)):
        ulps = np.abs(got.astype(np.longdouble) - want)[at] / np.spacing(want[at].astype(np.float64))
        assert float(ulps.max()) <= 1.3 and float(np.sqrt((ulps * ulps).mean())) <= 0.38, (float(ulps.max()), float(np.sqrt((ulps * ulps).mean())))


# lengths that leave some threads none; log-ratios on both sides of the 700
# from which the library exponential is taken, infinite and undefined ones among ordinary ones of the same wavefront
@pytest.mark.parametrize("lens", [[100, 128, 1], [130, 700, 257], [900, 1100, 255, 1025], [5000, 2049, 4096, 3]])
def test_objective_exponentials_by_rollout_length(A, lens):
    print("[case] grpo_objective exponentials %s" % lens, flush=True)
    rng = np.random.default_rng(sum(lens))
    T, beta = sum(lens), 0.04
    cu = np.concatenate([[0], np.cumsum(lens)])
    ref = (rng.normal(size=T) * 0.2).astype(np.float32)
    ref[rng.random(T) < 0.02] = 0.0
    odd = np.array([699.9, 700.0, 700.1, -699.9, -700.0, -700.1, 745.0, -745.0, 800.0, -800.0, np.inf, -np.inf, np.nan], np.float32)
    at = rng.choice(T, 26, replace=False)
    ref[at] = np.tile(odd, 2)
    adv = rng.normal(size=len(lens)).astype(np.float32)
    ws = torch.empty(16 * len(lens), dtype=torch.uint8, device=DEV)          # room for one part a rollout
    J, grad, n_clip = A.arrol_grpo_objective(torch.zeros(T, device=DEV), to_dev(ref, DEV), dev_i64(cu), to_dev(adv, DEV),
                                             torch.full((len(lens),), 1.0, device=DEV), 0.2, 0.28, beta, workspace=ws)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        u, a, scale = ref.astype(np.float64), np.repeat(adv.astype(np.float64), lens), np.repeat(1.0 / np.array(lens), lens)
        ratio, eu = np.exp(-u), np.exp(u)
        plain, clamped = ratio * a, np.fmin(np.fmax(ratio, 1.0 - f32(0.2)), 1.0 + f32(0.28)) * a
        want = ((np.where(plain <= clamped, plain, 0.0) - f32(beta) * (1.0 - eu)) * scale).astype(np.float32)
    got = npy(grad)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    ok = np.isfinite(want)
    # both exponentials within 2 ulp (4.4e-16 of terms of about 1 that cancel near u = 0), then one rounding to fp32
    assert np.all(np.abs(got[ok] - want[ok]) <= 1e-7 * np.abs(want[ok]) + 1e-15 * scale[ok] * 4)
    assert int(n_clip) == int(np.sum(clamped < plain)) and np.isnan(float(J))
    ref[at] = 0.1
    J = A.arrol_grpo_objective(torch.zeros(T, device=DEV), to_dev(ref, DEV), dev_i64(cu), to_dev(adv, DEV),
                               torch.full((len(lens),), 1.0, device=DEV), 0.2, 0.28, beta, workspace=ws)[0]
    u = ref.astype(np.float64); ratio, eu = np.exp(-u), np.exp(u)
    terms = (np.minimum(ratio * a, np.clip(ratio, 1.0 - f32(0.2), 1.0 + f32(0.28)) * a) - f32(beta) * (eu - u - 1.0)) * scale
    assert abs(float(J) - terms.sum()) <= 4e-15 * np.abs(terms).sum()


# rollouts cut into parts: lengths around the 1,024 tokens of a part, none, and far more than the mean; the workspace that
# decides how many parts there are (1, 2, 3 and the 8 the binding makes room for); the same bits again
@pytest.mark.parametrize("room", [1, 2, 3, 8])
def test_objective_in_parts(A, room):
    print("[case] grpo_objective parts room=%d" % room, flush=True)
    lens = [4096, 1, 0, 1023, 1024, 1025, 5000, 2049, 3, 8191, 4100, 2048]
    run_objective(A, lens, [4, 2, 6], seed=21, eps_high=0.28, beta=0.01)
    T, n = sum(lens), len(lens)
    g = torch.Generator(device=DEV); g.manual_seed(room)
    ref = -torch.rand(T, generator=g, device=DEV) * 4
    lp = ref + 0.3 * torch.randn(T, generator=g, device=DEV)
    adv, wgt, cu = torch.randn(n, generator=g, device=DEV), torch.rand(n, generator=g, device=DEV), dev_i64(np.concatenate([[0], np.cumsum(lens)]))
    whole = A.arrol_grpo_objective(lp, ref, cu, adv, wgt, beta=0.01)
    ws = torch.empty(16 * n * room, dtype=torch.uint8, device=DEV)
    part, again = (A.arrol_grpo_objective(lp, ref, cu, adv, wgt, beta=0.01, workspace=ws) for _ in range(2))
    torch.cuda.synchronize()
    assert torch.equal(whole[1], part[1]) and torch.equal(whole[2], part[2])      # per token: no sum in it
    # sums of T fp64 terms in another order
    assert abs(float(whole[0]) - float(part[0])) <= 1e-12 * max(1.0, abs(float(whole[0])))
    assert all(torch.equal(a, b) for a, b in zip(part, again))


# rollouts of no group get zeros, whatever the outputs held: before the first offset, behind the last, none, all, between
# groups whose offsets fall (which leaves ranges that no group holds), in one launch and, of many rollouts, in two
@pytest.mark.parametrize("offsets,N", [([0, 8, 20], 20), ([5, 8, 20], 33), ([7, 7], 12), ([0], 9), ([-4, 3, 99], 50), ([10, 30, 5, 8, 60, 40, 44], 90),
                                       ([40, 10], 64), ([3, 70000], 80000), ([60, 90, 20], 70001)])
def test_advantage_outside_every_group_is_zero(A, offsets, N):
    print("[case] grpo_advantage outside N=%d" % N, flush=True)
    reward = torch.randn(N, device=DEV)
    junk = [torch.full((N,), float("nan"), device=DEV) for _ in range(4)]
    del junk
    adv, wgt = A.arrol_grpo_advantage(reward, dev_i64(offsets))
    torch.cuda.synchronize()
    held = np.zeros(N, bool)
    for a, b in zip(offsets, offsets[1:]):
        a = min(max(a, 0), N)
        held[a:max(a, min(b, N))] = True
    assert np.all(npy(adv)[~held] == 0.0) and np.all(npy(wgt)[~held] == 0.0)
    assert np.all(npy(wgt)[held] > 0.0) and not np.isnan(npy(adv)).any()


# both sides of the bounds of the one launch (2,048 groups, 65,536 rollouts), offsets that rise, that hold few rollouts and of
# which one falls: no order of the offsets may make the call slow (some 25 us here; one wavefront that asked every group about
# every rollout took 22 ms at 16,384 x 1,024)
@pytest.mark.parametrize("kind", ["rise", "few", "fall"])
@pytest.mark.parametrize("N,n_groups", [(16384, 1024), (65536, 2048), (65537, 2048), (65536, 2049), (63, 1500), (129, 1), (1000, 513)])
def test_advantage_of_any_order_of_offsets(A, N, n_groups, kind):
    print("[case] grpo_advantage offsets %s N=%d groups=%d" % (kind, N, n_groups), flush=True)
    offsets = np.linspace(0, N, n_groups + 1).astype(np.int64)
    if kind == "few":
        offsets = N // 2 + offsets // 8
    elif kind == "fall":
        offsets = offsets // 2
        offsets[(n_groups + 1) // 2] = 1
    reward, off = torch.randn(N, device=DEV), dev_i64(offsets)
    adv, wgt = A.arrol_grpo_advantage(reward, off)
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    start.record()
    adv, wgt = A.arrol_grpo_advantage(reward, off)
    end.record()
    torch.cuda.synchronize()
    assert start.elapsed_time(end) < 10.0
    held = np.zeros(N, bool)
    for a, b in zip(offsets, offsets[1:]):
        held[a:max(a, min(b, N))] = True
    assert np.all(npy(adv)[~held] == 0.0) and np.all(npy(wgt)[~held] == 0.0)
    assert np.all(npy(wgt)[held] > 0.0) and not np.isnan(npy(adv)).any()
