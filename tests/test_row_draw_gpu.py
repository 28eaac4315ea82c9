"""GPU parity of the draw at T > 0 with whole rows in registers, and of the
row weight tables, against the oracle: rows at the edges of the vectors per
lane, rows without a finite maximum, values the tables lack, commits."""
import numpy as np
import pytest

from gpu_helpers import (assert_match, gpu_stages, gpu_step, oracle_step, say, to_device,
                         with_temperature)
from test_loop_gpu import GpuLoop, oracle_loop, widen
from test_parity_gpu import AUTO, FUSED, custom_case, workspace_left_clean
from paper_2609_20186_amd.workloads import f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_20186_amd import binding  # noqa: F401


# 1024 * 8 logits per vector and lane: kernels of 4, 8, 12, 16 and 20 vectors
# (two work-groups per unit with 4, hence more rows)
ROWS = {
    "v8": dict(seed=200, B=130, R=6, k=5, V=8, ties=True),
    "4_vectors": dict(seed=201, B=128, R=6, k=5, V=32768),
    "8_vectors": dict(seed=202, B=64, R=6, k=5, V=32776),
    "8_vectors_negative": dict(seed=203, B=64, R=6, k=5, V=33000, neg=True),
    "8_vectors_specials": dict(seed=204, B=64, R=6, k=5, V=40000, specials=True),
    "12_vectors_tree": dict(seed=205, B=13, R=32, k=7, V=65544, tree=True),
    "16_vectors": dict(seed=206, B=64, R=6, k=5, V=98312),
    "20_vectors": dict(seed=207, B=64, R=6, k=5, V=131080),
    "20_vectors_full": dict(seed=208, B=16, R=24, k=5, V=163840),
    "too_wide": dict(seed=209, B=64, R=6, k=5, V=163848),
    "many_sequences": dict(seed=210, B=256, R=4, k=3, V=520),
    "past_64_nodes": dict(seed=211, B=8, R=101, k=20, V=9000, n_cand=5),
}


@pytest.mark.parametrize("T", [0.7])
@pytest.mark.parametrize("case", sorted(ROWS))
def test_row_draw_parity(case, T):
    say(f"[row-draw] {case}")
    c = dict(ROWS[case])
    d = with_temperature(custom_case(Lmax=200, lens=(3, 2, 1), kappa=1, theta=0.0, vocab=6,
                                     plant=not c.get("neg") and not c.get("ties"), **c), T,
                         seed=300 + c["seed"])
    exp = oracle_step(d)
    dev = to_device(d)
    for mode in (AUTO, FUSED):
        got, ws = gpu_step(dev, d, mode)
        assert_match(got, exp, what=f"{case} mode {mode}")
        assert workspace_left_clean(ws, d)
    stages, _ = gpu_stages(dev, d)
    assert_match(stages, exp, what=f"{case} stages")


@pytest.mark.parametrize("B,R,V", [(64, 6, 33000), (32, 8, 128256)])
def test_values_below_the_table(B, R, V):
    """Most logits far smaller than the weight table's first entry, some zero,
    -inf or a negative NaN, a few ordinary: the vectors the table cannot serve
    are computed directly, in the row draw and in the sum launch."""
    say(f"[row-draw] small values {B}x{R}x{V}")
    d = custom_case(seed=220, B=B, Lmax=100, V=V, R=R, k=R - 1, lens=(2, 1), kappa=1, theta=0.0,
                    vocab=6)
    rng = np.random.default_rng(221)
    lg = d["logits"]
    small = rng.random(lg.shape) < 0.7
    lg[small] = (lg[small] & 0x807F) | (rng.integers(80, 112, int(small.sum())) << 7).astype(
        np.uint16)
    m = rng.random(lg.shape) < 0.01
    lg[m] = rng.choice(np.array([0x0000, 0x8000, 0xFF80, 0xFFC0, 0x0001], np.uint16),
                       int(m.sum()))
    d = with_temperature(d, 0.7, seed=222)
    exp = oracle_step(d)
    got, ws = gpu_step(to_device(d), d, AUTO)
    assert_match(got, exp, what="small values")
    assert workspace_left_clean(ws, d)


def test_row_draw_commits():
    """Decode steps with the commit inside the row draw's epilogue."""
    say("[row-draw] commit")
    d = with_temperature(custom_case(seed=230, B=64, Lmax=300, V=33000, R=6, k=5,
                                     lens=(3, 2, 1), kappa=1, theta=-0.3, vocab=6, plant=True),
                         0.6, seed=231)
    d = widen(d, 20)
    outs, tokens, lengths, draft_pos, lag = oracle_loop(d, 3)
    g = GpuLoop(d, AUTO)
    for _ in range(3):
        g.step()
    gt, gl, gd, glag = g.state()
    np.testing.assert_array_equal(gl, lengths)
    np.testing.assert_array_equal(gt, tokens)
    np.testing.assert_array_equal(gd, draft_pos)
    np.testing.assert_array_equal(glag, lag)


def pooled_logits(rng, B, R, V):
    """N(0, 1) rows cut from one pool at random places (fast for many rows)."""
    pool = f32_to_bf16_bits(np.clip(rng.standard_normal(V + (1 << 20)), -7.5, 7.5)
                            .astype(np.float32))
    out = np.empty((B, R, V), np.uint16)
    for row in out.reshape(B * R, V):
        at = int(rng.integers(0, 1 << 20))
        row[:] = pool[at:at + V]
    return out


def verify_sampled(d, dn, T):
    """switchsd_verify_sample over given drafts; the outputs, and whether the
    rows were drawn without the weight sums (their space stays as it was: only
    the maxima and sum launches write it)."""
    import torch
    from paper_2609_20186_amd import binding as sd
    B, R, V = d["logits"].shape
    dev = to_device(d)
    o = sd.alloc_outputs(B, R, d["cfg"]["k"])
    ws = sd.alloc_workspace(B, R, 1, 1)
    sws = sd.alloc_sample_workspace(B, R, V).fill_(0x5A)
    sd.switchsd_verify_sample(dev["logits"], T, dev["uniforms"], dev["ntok"], dev["npar"],
                              torch.from_numpy(dn).cuda(), o["accept_len"], o["accept_node"],
                              o["bonus"], o["out_tokens"], o["amax"], ws, sws)
    torch.cuda.synchronize()
    assert int(ws.count_nonzero()) == 0, "workspace not left zeroed"
    return o, bool((sws == 0x5A).all())


# where the row draw is the slower of the two: short rows (its kernels take a
# row's chain of steps, however short the row), rows that fill half a kernel's
# registers, too few rows
PATHS = {
    "tiny_rows": (130, 6, 8, False), "short_rows": (96, 13, 8000, False),
    "many_short_rows": (64, 64, 12000, False), "half_filled": (64, 20, 33000, False),
    "few_rows": (8, 8, 128256, False), "past_20_vectors": (48, 8, 163848, False),
    "3_chunks": (96, 13, 20000, True), "4_vectors": (96, 8, 32768, True),
    "7_chunks": (64, 8, 50000, True), "16_vectors": (48, 8, 128256, True),
    "long_drafts": (4, 201, 32000, True),
}


@pytest.mark.parametrize("case", sorted(PATHS))
def test_which_draw_is_taken(case):
    say(f"[row-draw] path {case}")
    import torch
    B, R, V, row = PATHS[case]
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 compute units")
    rng = np.random.default_rng(240)
    d = dict(logits=pooled_logits(rng, B, R, V), ntok=rng.integers(0, 6, (B, R)).astype(np.int32),
             npar=None, cfg=dict(k=R - 1), nn=np.full(B, R, np.int32), T=0.7, bias=0.0,
             uniforms=rng.integers(0, 2 ** 64, (B, R), dtype=np.uint64),
             tokens=np.zeros((B, 1), np.int32), lengths=np.ones(B, np.int32),
             hidden=np.zeros((B, 8), np.uint16), w=np.zeros(8, np.float32))
    dn = np.full(B, min(R, 8) if R > 64 else R, np.int32)
    _, by_rows = verify_sampled(d, dn, 0.7)
    assert by_rows == row
