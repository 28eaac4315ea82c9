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


# Rows at the edges of the row draw's kernels (8192 logits for each vector of a
# 1024-thread work-group); the shortest rows, and those just past 32768, are
# drawn from the weight sums (test_which_draw_is_taken)
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


def pooled_logits(rng, B, R, V, specials=False):
    """N(0, 1) rows cut from one pool at random places (fast for many rows).
    ``specials``: some rows negative throughout, all -inf, all NaN, with +inf or
    with NaN of either sign and zeros among ordinary values."""
    pool = f32_to_bf16_bits(np.clip(rng.standard_normal(V + (1 << 20)), -7.5, 7.5)
                            .astype(np.float32))
    out = np.empty((B, R, V), np.uint16)
    for row in out.reshape(B * R, V):
        at = int(rng.integers(0, 1 << 20))
        row[:] = pool[at:at + V]
        kind = int(rng.integers(0, 20)) if specials else 20
        if kind < 3:
            row |= np.uint16(0x8000)
        elif kind < 6:
            row[:] = (0xFF80, 0xFFC0, 0x7FC0)[kind - 3]
        elif kind == 6:
            row[rng.integers(0, V, 3)] = 0x7F80
        elif kind == 7:
            row[rng.integers(0, V, V // 8)] = rng.choice(
                np.array([0x7FC1, 0xFFC0, 0x0000, 0x8000, 0xFF80], np.uint16), V // 8)
    return out


def many_rows(rng, B, R, V, T, specials=False, tree=False):
    """Neural drafts of R rows for every sequence, part of each accepted."""
    npar = None
    if tree:
        npar = np.array([[-1] + [int(rng.integers(0, i)) for i in range(1, R)]
                         for _ in range(B)], np.int32)
    d = dict(logits=pooled_logits(rng, B, R, V, specials),
             ntok=rng.integers(0, min(V, 9), (B, R)).astype(np.int32), npar=npar,
             cfg=dict(lens=(2, 1), kappa=1, k=min(R - 1, 20), theta=1e9),
             nn=np.full(B, R, np.int32), T=T, bias=0.0,
             uniforms=rng.integers(0, 2 ** 64, (B, R), dtype=np.uint64),
             tokens=rng.integers(0, V, (B, 40)).astype(np.int32), lengths=np.full(B, 40, np.int32),
             hidden=np.zeros((B, 8), np.uint16), w=np.zeros(8, np.float32))
    # the drawn tokens do not depend on the draft: propose them as children
    # along part of each draft
    drawn = oracle_step(d)["amax"]
    par = np.arange(-1, R - 1)[None].repeat(B, 0) if npar is None else npar
    at = rng.random((B, R)) < 0.6
    at[:, 0] = False
    bi = np.arange(B)[:, None]
    d["ntok"] = np.where(at, drawn[bi, np.maximum(par, 0)], d["ntok"]).astype(np.int32)
    return d, oracle_step(d)


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


# four or more rows for every work-group of each of the row draw's kernels
# (512 of up to 32768 logits, else 256), ordinary rows between rows without a
# finite maximum; T = 30 makes no weight table (the table would lack most
# values).  sums_direct and streamed_sums_direct take the sum launches, whose
# rows have no table then either.
ROUNDS = {
    "512_threads": (128, 16, 16392, 0.7, True, False),
    "512_threads_long_drafts": (16, 201, 9000, 0.7, True, True),
    "8_vectors": (64, 16, 49160, 0.7, True, False),
    "8_vectors_direct": (64, 16, 49160, 30.0, True, False),
    "12_vectors_tree": (16, 64, 65544, 0.9, True, True),
    "16_vectors": (64, 16, 98312, 0.7, True, False),
    "20_vectors": (64, 16, 131080, 0.7, True, False),
    "20_vectors_direct": (32, 16, 131080, 25.0, True, False),
    "sums_direct": (64, 20, 33000, 30.0, False, False),
    "streamed_sums_direct": (2, 201, 163848, 30.0, False, True),
}


@pytest.mark.parametrize("case", sorted(ROUNDS))
def test_many_rounds(case):
    say(f"[row-draw] rounds {case}")
    import torch
    from paper_2609_20186_amd import binding as sd
    B, R, V, T, row, tree = ROUNDS[case]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    d, exp = many_rows(np.random.default_rng(250), B, R, V, T, specials=True, tree=tree)
    assert (exp["dn"] == R).all() and exp["accept_len"].mean() > 0.3
    sws = sd.alloc_sample_workspace(B, R, V).fill_(0x5A)
    got, ws = gpu_step(to_device(d), d, AUTO, sws=sws)
    assert_match(got, exp, what=case)
    assert workspace_left_clean(ws, d)
    o, by_rows = verify_sampled(d, exp["dn"], T)
    for k in ("amax", "accept_len", "accept_node", "bonus", "out_tokens"):
        np.testing.assert_array_equal(o[k].cpu().numpy(), exp[k], err_msg=k)
    if cus == 256:
        assert by_rows == row and bool((sws == 0x5A).all()) == row


def test_row_draw_commits_long_drafts():
    """Decode steps with the commit, drafts of ten copy candidates: several rows
    a work-group, the sequences closed after its last."""
    say("[row-draw] commit, long drafts")
    d = with_temperature(custom_case(seed=260, B=24, Lmax=600, V=8200, R=201, k=20,
                                     lens=(3, 2, 1), kappa=1, theta=-0.3, vocab=9, n_cand=10,
                                     plant=True, ragged=False), 0.6, seed=261)
    d["nn"][:] = 201
    d = widen(d, 80)
    outs, tokens, lengths, draft_pos, lag = oracle_loop(d, 3)
    assert outs[0]["dn"].sum() > 4 * 512 and 0 < outs[0]["use_copy"].sum() < 24
    g = GpuLoop(d, AUTO)
    g.sws.fill_(0x5A)
    for s in range(3):
        g.step()
        assert_match({k: v.cpu().numpy() for k, v in g.out.items()}, outs[s], what=f"step {s}")
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert bool((g.sws == 0x5A).all())
    gt, gl, gd, glag = g.state()
    np.testing.assert_array_equal(gl, lengths)
    np.testing.assert_array_equal(gt, tokens)
    np.testing.assert_array_equal(gd, draft_pos)
    np.testing.assert_array_equal(glag, lag)
