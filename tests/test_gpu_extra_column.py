"""GPU tests of the (d+1)-th column of the bucket statistics in the MFMA family: the masses A, which the matrix cores add up
from the bf16 assignments with weights of one, and their cotangents dA, whose fp32 weights enter as three bf16 parts."""
import numpy as np
import pytest
import torch

import paper_2510_04008_amd as ra
from paper_2510_04008_amd import synth
from paper_2510_04008_amd.synth import Workload

from parity_util import TOL, ErrAcc, desc_of, oracle_backward, oracle_forward, run_gpu, to_f64

pytestmark = pytest.mark.gpu

# every split of the bucket rows over the wavefronts: eight tables of 64, 16 of 16, four of 16 (two wavefronts a table), padded
SHAPES = [(128, 8, 6), (64, 16, 4), (128, 4, 4), (64, 5, 5), (128, 7, 3)]
# one token, around a tile of 32 and a step of 64, several segments, more segments than groups that add them up
LENGTHS = [1, 31, 33, 64, 95, 300, 2300]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("N", LENGTHS)
def test_masses_are_the_sums_of_the_assignments(shape, N):
    d, L, P = shape
    w = Workload("mass", 1, 2, N, d, L, P, 2.0, True, "bf16", normalize_qk=True, chunk=96)
    _, K, V, _ = synth.make_inputs(w, "cuda")
    seeds, desc = synth.projection_seeds(w), desc_of(w)
    assert ra.race_attn_kernel_family(desc) == 2
    _, phi = ra.race_attn_debug_hash(desc, K, seeds, want_phi=True)
    A, _ = ra.race_attn_debug_buckets(desc, K, V, seeds)
    ref = to_f64(phi).sum(axis=2)                                   # (B, H, L, R)
    # N positive terms in fp32, in any order: N roundings at most
    assert (np.abs(to_f64(A) - ref) <= N * 2.0 ** -24 * ref).all()


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_masses_of_a_long_segment_are_rounded_to_nearest(shape):
    """One segment of 524288 tokens: the masses that the accumulation alone forms, and those that the forward pass carries along,
    read by queries of zeros (whose assignments are 2^-P, exactly)."""
    d, L, P = shape
    w = Workload("long", 1, 1, 1 << 19, d, L, P, 2.0, True, "bf16", normalize_qk=True, chunk=1 << 19)
    Q, K, V, _ = synth.make_inputs(w, "cuda")
    Q = torch.zeros_like(Q)
    seeds, desc, last = synth.projection_seeds(w), desc_of(w), 256
    ref = torch.zeros((L << P,), dtype=torch.float64, device="cuda")
    for t0 in range(0, w.N, 1 << 15):
        part = K[:, :, t0:t0 + (1 << 15)].contiguous()
        _, phi = ra.race_attn_debug_hash(ra.make_desc(1, 1, 1 << 15, d, L, P, 2.0, True, ra.RACE_BF16), part, seeds, want_phi=True)
        phi = phi[0, 0].double().reshape(1 << 15, -1)
        ref += phi.sum(dim=0)
    A, _ = ra.race_attn_debug_buckets(desc, K, V, seeds)
    err = (A[0, 0].double().reshape(-1) - ref) / ref
    # two sums, of eight tokens in sixteen each, that grow evenly in n = N / 16 steps: a step is rounded to nearest, its error up to
    # 2^-24 of the sum so far, uniform (1 / sqrt 3) and independent, and the sum so far is 1 / sqrt 3 of the whole by root mean square
    rms = 2.0 ** -24 * (w.N / 32) ** 0.5 / 3
    off, mean = err.square().mean().sqrt().item(), err.mean().item()
    assert off <= rms, (off, mean)
    _, den = ra.race_attn_fwd(desc, Q, K, V, seeds)
    behind = phi[-last:].flip(0).cumsum(0).flip(0).sum(dim=1)       # mass of token i and those behind it
    want = (ref.sum() - torch.cat([behind[1:], behind.new_zeros(1)])) / (L << P)
    err = (den[0, 0, -last:].double() - want) / want
    # the same errors averaged over the bucket rows (four standard deviations), and the read-out's own sums
    most = err.abs().max().item()
    assert most <= 4 * rms / (L << P) ** 0.5 + 2.0 ** -22, most


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("causal", [True, False])
def test_gradient_through_the_cotangents_of_the_masses_alone(shape, causal):
    """With V = 0 the key side sees nothing but dA; O is an argument of the backward pass and is left as it is, and its rows are
    stretched over 2^-8 .. 2^8 so that the weights of one sum have very different sizes."""
    d, L, P = shape
    w = Workload("dA", 1, 2, 203, d, L, P, 2.0, causal, "bf16", normalize_qk=True, chunk=96)
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    stretch = torch.exp2(torch.arange(w.N, device="cuda") % 17 - 8.0)[None, None, :, None].to(torch.bfloat16)
    O_in, V = V * stretch, torch.zeros_like(V)
    _, den, ctx = oracle_forward(w, Q, K, V, synth.projection_seeds(w))
    den_in = torch.from_numpy(den).float().cuda()
    g = run_gpu(w, (Q, K, V, dO), fwd_results=lambda O, den: (O_in, den_in))
    _, dK, _ = oracle_backward(w, ctx, to_f64(O_in), to_f64(den_in), dO)
    acc = ErrAcc().update(g["dK"], dK)
    print("%s causal=%s: %s" % (shape, causal, acc), flush=True)
    assert acc.linf < TOL["bf16"] and acc.l2 < TOL["bf16"]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("bit", [10, 16])
def test_every_part_of_a_weight_counts(shape, causal, bit):
    """dA where all but the second (bit 10) or third (bit 16) eight bits of the weights cancel: queries come in pairs with the same
    row, hence the same assignments, and weights -s (1 + 2^-bit) and s.  Without those bits dA, and with V = 0 all of dK, is zero.
    Only the last 32 queries have cotangents, so that the keys in front of them meet fp32 statistics alone: those of earlier segments
    the scanned ones, those of earlier tiles of the same segment what the gradient kernel adds to them."""
    d, L, P = shape
    w = Workload("parts", 1, 2, 288, d, L, P, 2.0, causal, "bf16", normalize_qk=True, chunk=96)
    Q, K, V, _ = synth.make_inputs(w, "cuda")
    first = w.N - 32
    Q[:, :, first + 1::2] = Q[:, :, first::2]
    V, dO, O_in = torch.zeros_like(V), torch.zeros_like(V), torch.zeros_like(V)
    s = torch.tensor([1.0, -2.0, 0.5, -1.0, 4.0, 2.0, -0.25, -4.0, 1.0, 0.5, -2.0, 1.0, -0.5, 4.0, -1.0, 2.0], device="cuda").to(V.dtype)
    O_in[..., 0], O_in[..., 8] = 1.0, 2.0 ** -(bit // 2)
    dO[:, :, first::2, 0], dO[:, :, first::2, 8], dO[:, :, first + 1::2, 0] = s, s * 2.0 ** -(bit // 2), -s
    seeds = synth.projection_seeds(w)
    _, _, ctx = oracle_forward(w, Q, K, V, seeds)
    den_in = torch.full((1, 2, w.N), 1.0 / L, dtype=torch.float32, device="cuda")          # dO / (L Den) is dO itself
    g = run_gpu(w, (Q, K, V, dO), fwd_results=lambda O, den: (O_in, den_in))
    _, dK, _ = oracle_backward(w, ctx, to_f64(O_in), to_f64(den_in), dO)
    for part in (slice(0, 192), slice(192, first)):
        acc = ErrAcc().update(g["dK"][:, :, part], dK[:, :, part])
        print("%s causal=%s bit %d, keys %s: %s" % (shape, causal, bit, part, acc), flush=True)
        assert acc.linf < TOL["bf16"] and acc.l2 < TOL["bf16"]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_non_finite_key_has_finite_assignments(shape, unit, value):
    """... so that two tables that share a column of a matrix product cannot disturb one another."""
    d, L, P = shape
    w = Workload("key", 1, 1, 100, d, L, P, 2.0, True, "bf16", normalize_qk=True, chunk=96)
    _, K, V, _ = synth.make_inputs(w, "cuda")
    K2 = K.clone()
    K2[0, 0, 37, 5] = value
    desc = ra.make_desc(1, 1, w.N, d, L, P, 2.0, True, ra.RACE_BF16, 96, unit)
    seeds = synth.projection_seeds(w)
    _, phi = ra.race_attn_debug_hash(desc, K, seeds, want_phi=True)
    _, phi2 = ra.race_attn_debug_hash(desc, K2, seeds, want_phi=True)
    others = [i for i in range(w.N) if i != 37]
    assert torch.isfinite(phi2).all() and torch.equal(phi2[:, :, others], phi[:, :, others])
    A, B = ra.race_attn_debug_buckets(desc, K2, V, seeds)
    ref = phi2.double().sum(dim=2)
    assert torch.isfinite(B).all() and ((A.double() - ref).abs() <= w.N * 2.0 ** -24 * ref).all()
