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
