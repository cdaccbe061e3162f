"""The rows of Q and K are hashed either inside the forward's passes or by a kernel of their own in front of them, by a rule on the
number of workgroups and of their tiles.  Both run the same arithmetic: a batch that takes one way has, sequence by sequence and bit
for bit, the results of its sequences alone, which take the other; and both agree with the oracle at the edges of the tiles."""
import pytest
import torch

import paper_2510_04008_amd as ra
from paper_2510_04008_amd import synth
from paper_2510_04008_amd.synth import Workload

from parity_util import check_case, desc_of

pytestmark = pytest.mark.gpu

# exact and padded, one and several tables a half wavefront, tables shared by two of them
SHAPES = [(128, 8, 6), (64, 16, 4), (64, 6, 5), (64, 3, 2), (128, 12, 3), (128, 7, 3), (128, 4, 4)]


@pytest.mark.parametrize("causal,unit", [(True, False), (True, True), (False, False), (False, True)])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_both_ways_are_bit_identical(shape, causal, unit):
    d, L, P = shape
    # 6 tiles a workgroup, the last one ragged: not causal, 320 workgroups hash in the passes, 8 do not; causal, one segment, the kernel
    # hashes for both (several segments: below)
    B, H, N = 40, 8, 165
    w = Workload("rows", B, H, N, d, L, P, 4.0, causal, "bf16", chunk=192, unit_qk=unit)
    tensors = [t.cuda() if not t.is_cuda else t for t in synth.make_inputs(w, "cuda")]
    seeds = synth.projection_seeds(w)

    def run(desc, Q, K, V, dO):
        assert ra.race_attn_kernel_family(desc) == 2
        ws = torch.empty(ra.race_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        O, den = ra.race_attn_fwd(desc, Q, K, V, seeds, workspace=ws)
        grads = ra.race_attn_bwd_saved(desc, Q, K, V, O, den, dO, seeds, ws, want_dbeta=True)
        state = ra.race_attn_state_init(desc, K, V, seeds)
        torch.cuda.synchronize()
        return (O, den) + tuple(grads) + (state,)

    whole = run(desc_of(w), *tensors)
    one = desc_of(Workload("row", 1, H, N, d, L, P, 4.0, causal, "bf16", chunk=192, unit_qk=unit))
    for b in (0, B - 1):
        alone = run(one, *[t[b:b + 1].contiguous() for t in tensors])
        for name, x, y in zip(("O", "den", "dQ", "dK", "dV", "dbeta", "state"), whole, alone):
            assert torch.equal(x[b:b + 1], y), (name, b)


@pytest.mark.parametrize("N,chunk", [(31, 0), (97, 96), (128, 128), (129, 160), (300, 320)])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_tile_edges_against_the_oracle(shape, N, chunk):
    d, L, P = shape
    for causal in (True, False):
        check_case(Workload("rows-%d-%d" % (N, chunk), 1, 2, N, d, L, P, 2.0, causal, "bf16", normalize_qk=True, chunk=chunk), saved=True)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("N", [5, 32, 165])        # (of one token alone dQ and dK are zero, a difference of roundings)
@pytest.mark.parametrize("shape,dtype", [((128, 8, 6), "bf16"), ((64, 16, 4), "bf16"), ((128, 4, 4), "bf16"), ((32, 3, 3), "bf16"), ((64, 4, 4), "f32")], ids=str)
def test_one_segment_reads_nothing_that_was_not_written(shape, dtype, N, causal):
    # (a call of one segment leaves out the scans and, causal, the totals; the workspace is full of NaN)
    d, L, P = shape
    w = Workload("one", 1, 2, N, d, L, P, 2.0, causal, dtype, chunk=192, normalize_qk=True)
    check_case(w, saved=True)
    Q, K, V, dO = [t.cuda() for t in synth.make_inputs(w, "cuda")]
    seeds, desc, out = synth.projection_seeds(w), desc_of(w), []
    for fill in (0, 255):
        ws = torch.full((ra.race_attn_workspace_bytes(desc),), fill, dtype=torch.uint8, device="cuda")
        O, den = ra.race_attn_fwd(desc, Q, K, V, seeds, workspace=ws)
        out.append((O, den) + tuple(ra.race_attn_bwd_saved(desc, Q, K, V, O, den, dO, seeds, ws)))
    for x, y in zip(*out):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("shape", SHAPES + [(128, 6, 5)], ids=str)
def test_hashing_kernel_by_tiles_and_by_shares_of_a_tile(shape, unit):
    # eight sequences of 66 tiles, the last one ragged, of Q and K: a wavefront a tile; one of them: a wavefront a share of a tile
    d, L, P = shape
    w = Workload("shares", 8, 1, 2100, d, L, P, 2.0, True, "bf16", chunk=1056, unit_qk=unit)
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    seeds = synth.projection_seeds(w)

    def run(desc, *T):
        ws = torch.empty(ra.race_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        ra.race_attn_profile_enable(True)
        O, den = ra.race_attn_fwd(desc, T[0], T[1], T[2], seeds, workspace=ws)
        torch.cuda.synchronize()
        names = set(ra.race_attn_profile_read())
        ra.race_attn_profile_enable(False)
        assert "hash_rows" in names
        return (O, den) + tuple(ra.race_attn_bwd_saved(desc, T[0], T[1], T[2], O, den, T[3], seeds, ws))

    whole = run(desc_of(w), Q, K, V, dO)
    one = desc_of(Workload("share", 1, 1, 2100, d, L, P, 2.0, True, "bf16", chunk=1056, unit_qk=unit))
    for b in (0, 7):
        for x, y in zip(whole, run(one, *[t[b:b + 1].contiguous() for t in (Q, K, V, dO)])):
            assert torch.equal(x[b:b + 1], y), b


@pytest.mark.parametrize("causal,unit", [(True, False), (True, True), (False, False)])
@pytest.mark.parametrize("shape", SHAPES + [(128, 6, 5)], ids=str)
def test_both_ways_are_bit_identical_over_several_segments(shape, causal, unit):
    d, L, P = shape
    # three segments: five tiles (an odd one in the last 64-token step of the totals), five, and two, the last ragged, whose totals
    # nobody reads where the sequence is causal; 960 workgroups hash in the passes, 24 do not
    B, H, N = 40, 8, 357
    w = Workload("rows", B, H, N, d, L, P, 4.0, causal, "bf16", chunk=160, unit_qk=unit)
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    seeds = synth.projection_seeds(w)

    def run(desc, Q, K, V, dO, in_passes):
        ws = torch.empty(ra.race_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
        ra.race_attn_profile_enable(True)
        O, den = ra.race_attn_fwd(desc, Q, K, V, seeds, workspace=ws)
        torch.cuda.synchronize()
        names = set(ra.race_attn_profile_read())
        ra.race_attn_profile_enable(False)
        assert ("hash_rows" not in names) == in_passes and "stream_totals_kv" in names
        saved = ra.race_attn_bwd_saved(desc, Q, K, V, O, den, dO, seeds, ws, want_dbeta=True)
        again = ra.race_attn_bwd(desc, Q, K, V, O, den, dO, seeds)
        return (O, den) + tuple(saved) + tuple(again) + (ra.race_attn_state_init(desc, K, V, seeds),)

    whole = run(desc_of(w), Q, K, V, dO, True)
    one = desc_of(Workload("row", 1, H, N, d, L, P, 4.0, causal, "bf16", chunk=160, unit_qk=unit))
    for b in (0, B - 1):
        alone = run(one, *[t[b:b + 1].contiguous() for t in (Q, K, V, dO)], False)
        for name, x, y in zip(("O", "den", "dQ", "dK", "dV", "dbeta", "dQ recomputed", "dK recomputed", "dV recomputed", "state"), whole, alone):
            assert torch.equal(x[b:b + 1], y), (name, b)


@pytest.mark.parametrize("BH,N", [(8, 100), (256, 128), (320, 165)])
@pytest.mark.parametrize("shape", [(128, 8, 6), (64, 16, 4), (128, 4, 4)], ids=str)
def test_one_causal_segment_launches_no_totals_of_its_own(shape, BH, N):
    d, L, P = shape
    w = Workload("one", BH // 8, 8, N, d, L, P, 2.0, True, "bf16", chunk=192)
    Q, K, V, dO = synth.make_inputs(w, "cuda")
    seeds, desc = synth.projection_seeds(w), desc_of(w)
    ws = torch.empty(ra.race_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    launched = []
    O, den = ra.race_attn_fwd(desc, Q, K, V, seeds, workspace=ws)
    for call in (lambda: ra.race_attn_fwd(desc, Q, K, V, seeds, O, den, ws), lambda: ra.race_attn_bwd(desc, Q, K, V, O, den, dO, seeds, workspace=ws)):
        ra.race_attn_profile_enable(True)
        call()
        torch.cuda.synchronize()
        launched.append(set(ra.race_attn_profile_read()))
        ra.race_attn_profile_enable(False)
    assert launched == [{"hash_rows", "stream_forward"}, {"hash_rows", "stream_totals_qg", "stream_grad_v", "grad_q", "grad_k"}]


@pytest.mark.parametrize("shape,BH,N,chunk,in_passes", [
    ((64, 16, 4), 6, 6000, 0, True), ((128, 4, 4), 6, 6000, 0, True),           # a workgroup for nearly every CU
    ((128, 8, 6), 4, 1000, 128, False), ((128, 8, 6), 16, 1000, 128, True),     # four tiles each: 32 workgroups, 128
    ((128, 8, 6), 4, 1000, 64, True),                                           # two tiles each
    ((128, 8, 4), 36, 8192, 1024, False), ((128, 8, 4), 64, 8192, 1024, True),  # one round of workgroups and a bit, two rounds
], ids=str)
def test_where_rows_are_hashed(shape, BH, N, chunk, in_passes):
    d, L, P = shape
    w = Workload("where", 1, BH, N, d, L, P, 2.0, True, "bf16", chunk=chunk)
    Q, K, V, _ = synth.make_inputs(w, "cuda")
    desc = desc_of(w)
    ws = torch.empty(ra.race_attn_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    ra.race_attn_profile_enable(True)
    ra.race_attn_fwd(desc, Q, K, V, synth.projection_seeds(w), workspace=ws)
    torch.cuda.synchronize()
    names = set(ra.race_attn_profile_read())
    ra.race_attn_profile_enable(False)
    assert ("hash_rows" not in names) == in_passes
