"""GPU tests of infinities and NaNs in the generic kernels: in a causal sequence a token's value reaches itself and later
tokens only, and a read-out cotangent itself and earlier tokens only, also where it is not finite (a caller's padding, an
overflow elsewhere in a batch), and a query whose Den has underflowed to zero costs nobody else's gradients.  The reference
is the same call on finite inputs."""
import pytest
import torch

import paper_2510_04008_amd as ra
from paper_2510_04008_amd import synth
from paper_2510_04008_amd.synth import Workload

from parity_util import desc_of, run_gpu

pytestmark = pytest.mark.gpu

# room for the same sums in another order: some 32 terms of fp32 (bf16: one rounding of the result)
CLOSE = {"f32": 1e-5, "bf16": 2.0 ** -7}

# tiles of 16 tokens; of 32; narrow bf16; segments of several tiles; a table over several blocks; more than 128 columns
CASES = [Workload("nf16", 1, 2, 77, 64, 4, 4, 2.0, True, "f32", normalize_qk=True),
         Workload("nf32", 8, 8, 300, 32, 3, 3, 2.0, True, "f32", normalize_qk=True),
         Workload("nf-bf16", 1, 2, 77, 32, 4, 4, 2.0, True, "bf16", normalize_qk=True),
         Workload("nf-chunk", 1, 2, 200, 40, 2, 5, 2.0, True, "f32", normalize_qk=True, chunk=64),
         Workload("nf-wide", 2, 1, 70, 200, 1, 7, 2.0, True, "f32", normalize_qk=True)]


def _same(a, b, w):
    assert torch.isfinite(a).all()
    assert (a.double() - b.double()).abs().max().item() <= CLOSE[w.dtype] * b.double().abs().max().item()


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_non_finite_value_reaches_later_tokens_only(w, value):
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    ref = run_gpu(w, (Q, K, V, dO))
    assert ra.race_attn_kernel_family(desc_of(w)) == 1
    j, c = 41, 5                                         # neither first nor last of its tile
    V2 = V.clone()
    V2[0, 0, j, c] = value
    g = run_gpu(w, (Q, K, V2, dO), fwd_results=lambda O, den: (ref["O"], ref["den"]))
    cols = [i for i in range(w.d) if i != c]
    assert torch.equal(g["den"], ref["den"])
    _same(g["O"][0, 0, :j], ref["O"][0, 0, :j], w)
    _same(g["O"][..., cols], ref["O"][..., cols], w)
    assert not torch.isfinite(g["O"][0, 0, j:, c]).any()
    assert not torch.isfinite(g["dQ"][0, 0, j:]).all(dim=-1).any() and not torch.isfinite(g["dK"][0, 0, j]).any()
    _same(g["dQ"][0, 0, :j], ref["dQ"][0, 0, :j], w)
    _same(torch.cat([g["dK"][0, 0, :j], g["dK"][0, 0, j + 1:]]), torch.cat([ref["dK"][0, 0, :j], ref["dK"][0, 0, j + 1:]]), w)
    _same(g["dV"], ref["dV"], w)


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_non_finite_cotangent_reaches_earlier_tokens_only(w, value):
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    ref = run_gpu(w, (Q, K, V, dO))
    i, c = 38, 3
    dO2 = dO.clone()
    dO2[0, 0, i, c] = value
    g = run_gpu(w, (Q, K, V, dO2))
    cols = [e for e in range(w.d) if e != c]
    _same(g["dV"][0, 0, i + 1:], ref["dV"][0, 0, i + 1:], w)
    _same(g["dV"][..., cols], ref["dV"][..., cols], w)
    assert not torch.isfinite(g["dV"][0, 0, :i + 1, c]).any()
    _same(g["dK"][0, 0, i + 1:], ref["dK"][0, 0, i + 1:], w)
    _same(torch.cat([g["dQ"][0, 0, :i], g["dQ"][0, 0, i + 1:]]), torch.cat([ref["dQ"][0, 0, :i], ref["dQ"][0, 0, i + 1:]]), w)


@pytest.mark.parametrize("w", CASES + [Workload("nf-nc", 1, 2, 77, 64, 4, 4, 2.0, False, "f32", normalize_qk=True)], ids=lambda w: w.name)
def test_a_query_with_den_zero_contributes_no_gradient(w):
    # den = 0 comes with O = 0 (the buckets a query reads hold no mass that fp32 can express): a constant output
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    i = 38
    dO2 = dO.clone()
    dO2[0, 0, i] = 0
    ref = run_gpu(w, (Q, K, V, dO2))
    O, den = ref["O"].clone(), ref["den"].clone()
    O[0, 0, i] = 0
    den[0, 0, i] = 0
    g = run_gpu(w, (Q, K, V, dO), fwd_results=lambda O_, den_: (O, den))
    for n in ("dQ", "dK", "dV"):
        assert torch.isfinite(g[n]).all() and torch.equal(g[n], ref[n]), n
