"""The chunked kernel of fp32 tensors against the fp64 oracle where it can go wrong: chunk, round and column-group edges, sequences
that end inside a chunk, decays at both ends of their range, values that are not finite."""
import numpy as np
import pytest
import torch

import paper_2407_12077_amd as wkv
from gpu_util import TOL_F32, max_norm_err, run_entry
from oracle import wkv6_oracle

pytestmark = pytest.mark.gpu


def inputs(B, T, H, seed, state=True):
    rng = np.random.default_rng(seed)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    return {"r": f(B, T, H, 64) / 8, "k": f(B, T, H, 64) / 8, "v": f(B, T, H, 64) / 8,
            "x": rng.uniform(-6, 1, (B, T, H, 64)).astype(np.float32), "u": f(H, 64) / 2,
            "state_in": f(B, H, 64, 64) / 10 if state else None}


def run(inp, **kw):
    return run_entry("wkv6_prefill_f32", inp, in_dtype=torch.float32, **kw)


# one, two and four column blocks a workgroup (up to 64, 128 and more units), below and above 256 workgroups; tokens around a
# chunk (16), a round of four chunks (64), two rounds
@pytest.mark.parametrize("B,H", [(1, 3), (1, 25), (2, 32), (5, 13), (4, 32), (3, 43), (8, 32), (2, 129)])
@pytest.mark.parametrize("T", [97, 112, 113, 127, 128, 129, 145, 192, 193, 257])
def test_edges_of_chunks_and_rounds(B, H, T):
    inp = inputs(B, T, H, 100 * T + B * H, state=T % 2 == 0)
    o, s = run(inp)
    o_ref, s_ref = wkv6_oracle(**inp)
    assert max_norm_err(o, o_ref) <= TOL_F32 and max_norm_err(s, s_ref) <= TOL_F32


# scores from a kernel of their own: the shortest such sequences of few units, chunks that end inside, rounds of four chunks
@pytest.mark.parametrize("B,H,T", [(1, 1, 201), (1, 1, 202), (3, 1, 209), (2, 16, 264), (4, 8, 271), (32, 1, 319), (1, 64, 327), (1, 64, 328), (2, 32, 385), (1, 5, 1023)])
@pytest.mark.parametrize("state", [False, True])
def test_scores_handed_over_in_rows_of_out(B, H, T, state):
    inp = inputs(B, T, H, T, state)
    o, s = run(inp)
    o_ref, s_ref = wkv6_oracle(**inp)
    assert max_norm_err(o, o_ref) <= TOL_F32 and max_norm_err(s, s_ref) <= TOL_F32


@pytest.mark.parametrize("name,value", [("v", np.inf), ("k", np.nan), ("r", np.inf), ("x", np.nan)])
def test_a_value_that_is_not_finite_with_scores_handed_over(name, value):
    """What came before the value has the bits that it has without it."""
    inp = inputs(1, 320, 4, 5)
    inp["x"] = inp["x"].clip(-6, -1)
    clean = run(inp)
    inp[name][0, 231, 2, 37] = value
    o, s = run(inp)
    with np.errstate(all="ignore"):
        o_ref, s_ref = wkv6_oracle(**inp)
    for got, ref in ((o, o_ref), (s, s_ref)):
        assert (np.isfinite(got) == np.isfinite(ref)).all()
        assert max_norm_err(got[np.isfinite(ref)], ref[np.isfinite(ref)]) <= TOL_F32
    assert np.array_equal(o[0, :231], clean[0][0, :231])


@pytest.mark.parametrize("B,H,T", [(25, 1, 33), (25, 1, 48), (5, 16, 49), (100, 1, 24), (100, 1, 25), (200, 1, 24), (200, 1, 31), (300, 1, 48), (300, 1, 63)])
def test_shortest_sequences(B, H, T):
    inp = inputs(B, T, H, T)
    o, s = run(inp, inplace_state=True)
    o_ref, s_ref = wkv6_oracle(**inp)
    assert max_norm_err(o, o_ref) <= TOL_F32 and max_norm_err(s, s_ref) <= TOL_F32


@pytest.mark.parametrize("H", [4, 100, 200])
def test_error_is_that_of_fp32_sums(H):
    """Each output is a sum of some hundred products: 1.3e-7 relative to its 2-norm leaves a factor of 1.4 over 9.4e-8 (state 5.8e-8),
    which is what the token-by-token kernels show, and lies below the 1.6e-7 of one chain of sums per 64 products."""
    inp = inputs(1, 300, H, 7)
    o, s = run(inp)
    for got, ref in zip((o, s), wkv6_oracle(**inp)):
        assert np.linalg.norm(got - ref) <= 1.3e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("H", [4, 70, 130])
def test_decays_at_the_ends_of_their_range(H):
    inp = inputs(1, 200, H, 3)
    rng = np.random.default_rng(4)
    kind = rng.integers(0, 8, inp["x"].shape)
    for i, v in enumerate((np.inf, -np.inf, 40., -40., 100., -200.)):
        inp["x"][kind == i] = v
    o, s = run(inp)
    o_ref, s_ref = wkv6_oracle(**inp)
    assert max_norm_err(o, o_ref) <= TOL_F32 and max_norm_err(s, s_ref) <= TOL_F32


@pytest.mark.parametrize("H", [4, 70, 130])
@pytest.mark.parametrize("name,value", [("v", np.inf), ("v", np.nan), ("k", np.inf), ("r", -np.inf), ("x", np.nan), ("state_in", np.nan)])
def test_a_value_that_is_not_finite_reaches_only_what_depends_on_it(H, name, value):
    T, t0, h0, n0 = 130, 71, 2, 37
    inp = inputs(1, T, H, 9)
    inp["x"] = inp["x"].clip(-6, -1)                          # no decay product underflows: zero times infinity stays out of it
    clean = run(inp)
    if name == "state_in":
        inp[name][0, h0, n0, 5] = value
    else:
        inp[name][0, t0, h0, n0] = value
    o, s = run(inp)
    with np.errstate(all="ignore"):
        o_ref, s_ref = wkv6_oracle(**inp)
    for got, ref, before in ((o, o_ref, clean[0]), (s, s_ref, clean[1])):
        assert (np.isfinite(got) == np.isfinite(ref)).all()
        same = np.isfinite(ref)
        assert max_norm_err(got[same], ref[same]) <= TOL_F32
    assert np.array_equal(o[0, :t0, :, :] if name != "state_in" else o[0, :, :h0], clean[0][0, :t0] if name != "state_in" else clean[0][0, :, :h0])


@pytest.mark.parametrize("T", [200, 300])
def test_result_is_the_same_under_capture(T):
    B, H = 2, 16
    inp = inputs(B, T, H, 1)
    dev = {n: torch.from_numpy(np.ascontiguousarray(a)).cuda() for n, a in inp.items()}
    out, state = torch.empty_like(dev["r"]), torch.empty_like(dev["state_in"])
    call = lambda: wkv.wkv6_prefill_f32(B, T, H, 64, dev["r"], dev["k"], dev["v"], dev["x"], dev["u"], dev["state_in"], out, state)  # noqa: E731
    call()
    torch.cuda.synchronize()
    eager = out.clone(), state.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        out.zero_(), state.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager[0]) and torch.equal(state, eager[1])
