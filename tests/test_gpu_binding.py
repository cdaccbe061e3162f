"""GPU tests of the extension module that marshals the hot calls (csrc/native_binding.cpp): what it refuses, the forms of seeds
and streams it takes, and calls from two Python threads."""
import threading

import numpy as np
import pytest
import torch

import paper_2510_04008_amd as ra

pytestmark = pytest.mark.gpu

B, H, N, D, L, P = 1, 2, 200, 32, 2, 3


def _desc(n=N, causal=True):
    return ra.make_desc(B, H, n, D, L, P, 2.0, causal, ra.RACE_F32)


def _buffers(seed=0, device="cuda"):
    gen = torch.Generator().manual_seed(seed)
    t = {n: torch.randn((B, H, N, D), generator=gen).to(device) for n in ("Q", "K", "V", "dO")}
    t.update({n: torch.empty((B, H, N, D), device=device) for n in ("O", "dQ", "dK", "dV")})
    t["den"] = torch.empty((B, H, N), device=device)
    t["dbeta"] = torch.empty((B, H), device=device)
    t["ws"] = torch.empty(ra.race_attn_workspace_bytes(_desc()), dtype=torch.uint8, device=device)
    return t


def _fwd(t, seeds=(1, 2), stream=None, desc=None):
    return ra.race_attn_fwd(desc or _desc(), t["Q"], t["K"], t["V"], seeds, t["O"], t["den"], t["ws"], stream)


def _bwd(t, seeds=(1, 2), stream=None):
    return ra.race_attn_bwd_saved(_desc(), t["Q"], t["K"], t["V"], t["O"], t["den"], t["dO"], seeds, t["ws"], t["dQ"], t["dK"], t["dV"],
                                  t["dbeta"], stream=stream)


WRONG = {"shape": lambda t: torch.zeros(t.shape + (1,), dtype=t.dtype, device=t.device),
         "size": lambda t: torch.zeros(tuple(s + 1 for s in t.shape), dtype=t.dtype, device=t.device),
         "dtype": lambda t: t.to(torch.float16),
         "stride": lambda t: torch.zeros(t.shape[:-1] + (2 * t.shape[-1],), dtype=t.dtype, device=t.device)[..., ::2],
         "device": lambda t: t.cpu(),
         "type": lambda t: t.cpu().numpy()}


@pytest.mark.parametrize("how", WRONG)
def test_every_tensor_is_checked(how):
    for name in ("Q", "K", "V", "O", "den"):
        t = _buffers()
        t[name] = WRONG[how](t[name])
        with pytest.raises(ValueError):
            _fwd(t)
    for name in ("Q", "K", "V", "O", "den", "dO", "dQ", "dK", "dV", "dbeta"):
        t = _buffers()
        t[name] = WRONG[how](t[name])
        with pytest.raises(ValueError):
            _bwd(t)
    desc = _desc()
    for name in ("q", "k", "v", "state", "o", "den"):
        s = {n: torch.zeros((B, H, D), device="cuda") for n in ("q", "k", "v", "o")}
        s["den"] = torch.zeros((B, H), device="cuda")
        s["state"] = ra.race_attn_state_init(_desc(0), None, None, (1, 2))
        s[name] = WRONG[how](s[name])
        with pytest.raises(ValueError):
            ra.race_attn_step(desc, s["q"], s["k"], s["v"], (1, 2), s["state"], s["o"], s["den"],
                              torch.empty(ra.race_attn_step_workspace_bytes(desc), dtype=torch.uint8, device="cuda"))
        if name == "state":
            with pytest.raises(ValueError):
                ra.race_attn_state_init(_desc(0), None, None, (1, 2), state=s["state"])
    torch.cuda.synchronize()


def test_a_short_workspace_is_refused():
    t = _buffers()
    t["ws"] = t["ws"][:-256]
    with pytest.raises(ra.RaceAttnError) as e:
        _fwd(t)
    assert e.value.status == ra.RACE_ERR_WORKSPACE


@pytest.mark.parametrize("seeds", [[1.0, 2.0], (np.uint64(1), np.int32(2)), np.array([1, 2], dtype=np.uint64), torch.tensor([1, 2]),
                                   torch.tensor([1.0, 2.0]), [1 + (1 << 64), 2 - (1 << 64)], [1, 2, 3]],
                         ids=["float", "numpy", "array", "tensor", "float-tensor", "modulo", "more"])
def test_seeds_are_taken_as_numbers(seeds):
    ref = tuple(x.clone() for x in _fwd(_buffers()))
    for a, b in zip(_fwd(_buffers(), seeds), ref):
        assert torch.equal(a, b)


def test_missing_seeds_are_refused_where_they_are_read():
    t = _buffers()
    _fwd(t)
    for call in (_fwd, _bwd):
        with pytest.raises(ValueError):
            call(t, [1])
        with pytest.raises(TypeError):
            call(t, None)
        with pytest.raises(TypeError):
            call(t, [object(), 2])
    with pytest.raises(ValueError):
        ra.race_attn_state_init(_desc(), t["K"], t["V"], [1])
    with pytest.raises(TypeError):
        ra.race_attn_state_init(_desc(0), None, None, None)
    # an empty context reads none
    state = ra.race_attn_state_init(_desc(0), None, None, [])
    assert state.shape == (B, H, L, 1 << P, D + 1) and not state.any()
    empty = torch.empty((B, H, 0, D), device="cuda")
    O, den = ra.race_attn_fwd(_desc(0), empty, empty, empty, [])
    assert O.shape == empty.shape and den.shape == (B, H, 0)


def test_streams_may_be_objects_or_handles():
    ref = tuple(x.clone() for x in _fwd(_buffers()))
    side = torch.cuda.Stream()
    for stream in (side, side.cuda_stream, 0):
        t = _buffers()
        torch.cuda.synchronize()
        _fwd(t, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(t["O"], ref[0]) and torch.equal(t["den"], ref[1])
    with torch.cuda.stream(side):
        t = _buffers()
        _fwd(t)
    torch.cuda.synchronize()
    assert torch.equal(t["O"], ref[0])
    with pytest.raises((TypeError, ValueError)):
        _fwd(_buffers(), stream="main")


def test_two_python_threads():
    names = ("O", "den", "dQ", "dK", "dV", "dbeta")
    refs = []
    for i in range(2):
        t = _buffers(i)
        _fwd(t, (10 + i, 20 + i))
        _bwd(t, (10 + i, 20 + i))
        torch.cuda.synchronize()
        refs.append({n: t[n].clone() for n in names})
    errors = []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                t = _buffers(i)
                for _ in range(30):
                    _fwd(t, (10 + i, 20 + i))
                    _bwd(t, (10 + i, 20 + i))
                    for n in names:
                        assert torch.equal(t[n], refs[i][n]), n
        except BaseException as e:                      # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors
