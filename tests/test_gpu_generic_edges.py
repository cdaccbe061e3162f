"""GPU tests of the generic kernels where a block of 64 bucket rows, a row tile of 16 or a group of 16 hyperplanes is not full, a
table spans blocks, and the waves share the projection in every way (1, 2 and 4 tiles of 16 tokens x 16 hyperplanes a block)."""
import pytest
import torch

from paper_2510_04008_amd import synth
from paper_2510_04008_amd.synth import Workload

from parity_util import check_case, run_gpu

pytestmark = pytest.mark.gpu

# (B, H, N, d, L, P): 6, 12, 24 and 36 bucket rows; 27 hyperplanes in two groups; several blocks; a table over two blocks; the
# same with 32-token tiles (more than 1024 tiles of 16) and with segments of two tiles
CASES = [(1, 2, 45, 8, 3, 1), (1, 2, 45, 24, 3, 2), (1, 2, 45, 40, 3, 3), (1, 1, 77, 64, 9, 2), (1, 1, 33, 72, 27, 1), (1, 1, 45, 104, 3, 5),
         (1, 1, 45, 136, 2, 7), (8, 8, 300, 24, 3, 2), (8, 8, 300, 24, 27, 1), (8, 8, 1100, 8, 3, 2)]


@pytest.mark.parametrize("case,dtype", [(c, "f32") for c in CASES] + [(CASES[i], "bf16") for i in (0, 1, 2, 5, 6)], ids=str)
@pytest.mark.parametrize("causal", [True, False])
def test_parity(case, causal, dtype):
    B, H, N, d, L, P = case
    check_case(Workload("edges", B, H, N, d, L, P, 2.0, causal, dtype, normalize_qk=True), saved=True)


@pytest.mark.parametrize("case", CASES[:4], ids=str)
def test_an_infinity_stays_in_its_column(case):
    """Bucket rows that do not exist take no part in the read-out, not even as a zero times an infinity."""
    B, H, N, d, L, P = case
    w = Workload("inf", B, H, N, d, L, P, 2.0, False, "f32", normalize_qk=True)
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    ref = run_gpu(w, (Q, K, V, dO))
    V2 = V.clone()
    V2[0, 0, N - 1, 3] = float("inf")
    g = run_gpu(w, (Q, K, V2, dO), fwd_results=lambda O, den: (ref["O"], ref["den"]))
    cols = [c for c in range(d) if c != 3]
    assert torch.equal(g["O"][..., cols], ref["O"][..., cols]) and torch.equal(g["den"], ref["den"])
    assert (g["O"][0, 0, :, 3] == float("inf")).all()
    assert torch.equal(g["dV"], ref["dV"])


@pytest.mark.parametrize("case", CASES[:4], ids=str)
@pytest.mark.parametrize("causal", [True, False])
def test_an_infinite_cotangent_stays_in_its_column(case, causal):
    """The same for the read-out of the cotangent statistics: dV's column is an infinity, not the NaN of a zero times one."""
    B, H, N, d, L, P = case
    w = Workload("inf", B, H, N, d, L, P, 2.0, causal, "f32", normalize_qk=True)
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    ref = run_gpu(w, (Q, K, V, dO))
    i = N // 2
    dO2 = dO.clone()
    dO2[0, 0, i, 3] = float("inf")
    g = run_gpu(w, (Q, K, V, dO2))
    last = i + 1 if causal else N                                   # tokens whose value the query reads
    cols = [c for c in range(d) if c != 3]
    assert torch.equal(g["dV"][..., cols], ref["dV"][..., cols]) and torch.equal(g["dV"][0, 0, last:], ref["dV"][0, 0, last:])
    assert torch.equal(g["dV"][0, 1:], ref["dV"][0, 1:])
    assert (g["dV"][0, 0, :last, 3] == float("inf")).all()


@pytest.mark.parametrize("d", [72, 136, 200, 256])
@pytest.mark.parametrize("shape", [(1, 2, 45), (8, 8, 300)], ids=["tiles16", "tiles32"])
@pytest.mark.parametrize("L,P", [(3, 2), (9, 3)])
def test_wide_rows_take_their_hyperplanes_part_by_part(d, shape, L, P):
    """More than 64 columns: 6, 24 and 3 hyperplanes a block, i.e. one, two and four parts of a hyperplane's row per wavefront."""
    check_case(Workload("wide", *shape, d, L, P, 2.0, True, "f32", normalize_qk=True), saved=True)
