"""GPU parity of ResidualAttention chunked prefill against the fp64 CPU oracle.

Each agent appends a chunk (fkv_cow_append) and its chunk's query rows attend
causally to the shared prefix, the agent's own suffix and the chunk so far.
Same bar as decode: max abs <= 2e-2, mean abs <= 2e-3, plus relative L2 <= 1e-2.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_06370_amd import _native as N
from paper_2604_06370_amd import workloads as W
from paper_2604_06370_amd.driver import LoadedWorkload

pytestmark = pytest.mark.gpu

TOL_MAX, TOL_MEAN, TOL_REL = 2e-2, 2e-3, 1e-2


def check_close(tag, out_gpu, ref):
    g = out_gpu.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(g).all(), f"{tag}: non-finite output"
    err = np.abs(g - ref)
    rel = np.linalg.norm(g - ref) / max(np.linalg.norm(ref), 1e-30)
    print(f"[{tag}] max {err.max():.3e} mean {err.mean():.3e} relL2 {rel:.3e} |ref| {np.abs(ref).mean():.3e}",
          flush=True)
    assert err.max() <= TOL_MAX and err.mean() <= TOL_MEAN and rel <= TOL_REL, tag
    return g


def run_prefill(tag, wl, rope, q_sample=None, no_residual=False):
    print(f"case {tag}: agents={wl.n_agents} hq={wl.hq} hkv={wl.hkv} r={wl.r} rope={rope} "
          f"L={list(wl.seq_len[:4])} chunks={[len(c) for c in wl.chunk_tokens[:4]]}", flush=True)
    lw = LoadedWorkload(wl, rope=rope, no_residual=no_residual)
    st = lw.prefill_setup()
    out = lw.prefill().clone()
    torch.cuda.synchronize()
    agents = st["agents"]
    q_rows = None
    if q_sample is not None:
        q_rows = {a: q_sample(wl.n_queries(a)) for a in agents}
    p = W.oracle_inputs(wl, agents=agents, q_rows=q_rows, rope=rope)
    if no_residual:
        p["has_residual"] = np.zeros_like(p["has_residual"])
    ref = oracle.residual_attention(p)
    # map the oracle's rows back to the kernel's output rows
    rows = st["rows"]
    pos = {int(x): i for i, x in enumerate(rows)}
    sel = [pos[int(x)] for x in p["q_index"]]
    g = check_close(tag, out[sel], ref)
    return lw, g, ref


@pytest.mark.parametrize("rope", [False, True])
def test_prefill_small_ragged(rope):
    wl = W.fanout("pf-small", 51, n_agents=4, prefix=256, suffix_lo=5, suffix_hi=40, hq=32, hkv=8, r=16,
                  chunk=100, chunk_c_from_hidden=True)
    lw, g, ref = run_prefill(f"prefill-small rope={rope}", wl, rope)
    # residual delta against the base-only run
    lw0, g0, ref0 = run_prefill(f"prefill-small base-only rope={rope}", wl, rope, no_residual=True)
    dg, dr = g - g0, ref - ref0
    ratio = np.linalg.norm(dg - dr) / np.linalg.norm(dr)
    print(f"residual delta relerr {ratio:.3e} |d_ref| {np.abs(dr).mean():.3e}", flush=True)
    assert ratio <= 0.1


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("hq,hkv", [(12, 3), (16, 2)])
def test_prefill_other_head_layouts(rope, hq, hkv):
    """KV-head counts other than 8 (an odd one included) and eight query heads per KV head."""
    wl = W.fanout(f"pf-hq{hq}-hkv{hkv}", 59, n_agents=3, prefix=200, suffix_lo=1, suffix_hi=40, hq=hq, hkv=hkv,
                  r=16, chunk=90, b_std=0.25)
    run_prefill(f"prefill hq={hq} hkv={hkv} rope={rope}", wl, rope)


@pytest.mark.parametrize("rope", [False, True])
def test_prefill_70b_heads_rank64(rope):
    wl = W.tree("pf-70b", 52, node_parent=[-1, -1], node_len=[300, 700], agent_node=[0, 1, 0, 1],
                suffix_lo=1, suffix_hi=60, hq=64, hkv=8, r=64, b_std=0.05, chunk=[70, 33, 1, 129],
                zero_residual=[2])
    run_prefill(f"prefill-70b rope={rope}", wl, rope)


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("rank,hq", [(0, 32), (8, 32), (32, 32), (16, 64)])
def test_prefill_other_ranks(rank, hq, rope):
    wl = W.fanout(f"pf-r{rank}-hq{hq}", 53, n_agents=3, prefix=128, suffix_lo=1, suffix_hi=30, hq=hq, hkv=8,
                  r=max(rank, 8), chunk=64, zero_residual=range(3) if rank == 0 else ())
    run_prefill(f"prefill-r{rank}-hq{hq} rope={rope}", wl, rope)


@pytest.mark.parametrize("rope", [False, True])
def test_prefill_single_tile_and_one_token_chunks(rope):
    """Sequences of one 64-key tile or less (no copy runs ahead) and chunks of one token."""
    wl = W.fanout("pf-tiny", 56, n_agents=3, prefix=8, suffix_lo=0, suffix_hi=20, hq=32, hkv=8, r=16, chunk=30)
    run_prefill(f"prefill-one-tile rope={rope}", wl, rope)
    wl1 = W.fanout("pf-one", 57, n_agents=2, prefix=100, suffix_lo=0, suffix_hi=3, hq=32, hkv=8, r=16, chunk=1)
    run_prefill(f"prefill-one-token rope={rope}", wl1, rope)


def test_copy_on_write_at_fork_and_append():
    """Three agents fork the same 500-token context (the last page is partial and shared
    read-only), then each appends its own chunk: the first two appends copy the shared
    page (copy-on-write), the third writes in place.  A fourth agent forks 500 shared
    tokens plus its own suffix and copies 4 tokens of the partial page at fork time."""
    wl = W.fanout("cow", 54, n_agents=3, prefix=500, suffix_lo=0, suffix_hi=0, hq=32, hkv=8, r=16,
                  chunk=37, fixed_suffix=0)
    lw, g, ref = run_prefill("cow-append", wl, True)
    base_copies = [c for fp in lw.append_plans for c in fp.copies if c[0] == 0]
    assert len(base_copies) == 2 and all(c[3] == 4 for c in base_copies)
    wl2 = W.fanout("cow-fork", 55, n_agents=4, prefix=500, suffix_lo=3, suffix_hi=40, hq=32, hkv=8, r=16)
    lw2 = LoadedWorkload(wl2, rope=True)
    fork_copies = [c for fp in lw2.fill_plans for c in fp.copies if c[0] == 0]
    assert len(fork_copies) == 3 and all(c[3] == 4 for c in fork_copies)
    out = lw2.decode().clone()
    torch.cuda.synchronize()
    ref2 = oracle.residual_attention(W.oracle_inputs(wl2, rope=True))
    check_close("cow-fork decode", out, ref2)


@pytest.mark.parametrize("rope", [False, True])
def test_config3_full_size_sampled(rope):
    """Config 3 at full size: 16 agents append 2048-token chunks after a 32768-token shared
    prefix and a private suffix; rows are sampled (first, last, and random ones) for three
    agents and compared with the oracle."""
    wl = W.config(3)
    rng = np.random.default_rng(9)
    lw = LoadedWorkload(wl, rope=rope)
    st = lw.prefill_setup()
    out = lw.prefill().clone()
    torch.cuda.synchronize()
    agents = [0, 5, 15]
    q_rows = {a: np.unique(np.concatenate([[0, 1, 63, 64, 2047], rng.integers(0, 2048, 5)])) for a in agents}
    p = W.oracle_inputs(wl, agents=agents, q_rows=q_rows, rope=rope)
    ref = oracle.residual_attention(p)
    pos = {int(x): i for i, x in enumerate(st["rows"])}
    check_close(f"cfg3-full rope={rope}", out[[pos[int(x)] for x in p["q_index"]]], ref)
    lw.close()


@pytest.mark.parametrize("rope", [False, True])
def test_config5_mixed_full_size_sampled(rope):
    """Config 5 at full size: 32 agents of a 70B-shaped layer (64 q / 8 kv heads, rank 64) over
    three trees (8K / 32K / 64K prefixes), agents i mod 10 == 9 without residual; 8 agents
    prefill a 1024-token chunk and 24 decode, both calls on one stream.  Sampled decode agents
    cover every tree and a zero-residual agent; sampled prefill rows cover three agents."""
    wl = W.config(5)
    print(f"case cfg5-full rope={rope}: agents={wl.n_agents} L={list(wl.seq_len[:6])}...", flush=True)
    lw = LoadedWorkload(wl, rope=rope)
    dec_agents = wl.decode_agents()
    st = lw.prefill_setup()
    out_d = lw.decode().clone()
    out_p = lw.prefill().clone()
    torch.cuda.synchronize()
    dsample = [0, 1, 2, 9, 29]
    p = W.oracle_inputs(wl, agents=dsample, rope=rope)
    ref = oracle.residual_attention(p)
    check_close(f"cfg5-decode rope={rope}", out_d[[dec_agents.index(a) for a in dsample]], ref)
    rng = np.random.default_rng(11)
    pagents = [3, 19, 23]
    q_rows = {a: np.unique(np.concatenate([[0, 1, 15, 16, 1023], rng.integers(0, 1024, 5)])) for a in pagents}
    p = W.oracle_inputs(wl, agents=pagents, q_rows=q_rows, rope=rope)
    ref = oracle.residual_attention(p)
    pos = {int(x): i for i, x in enumerate(st["rows"])}
    check_close(f"cfg5-prefill rope={rope}", out_p[[pos[int(x)] for x in p["q_index"]]], ref)
    lw.close()


def test_understated_row_count_shows_as_nan_rows():
    """max_q_per_agent sizes the grid; rows of an agent beyond what it covers are not computed
    and must come out as NaN (never stale memory), while the covered rows stay correct."""
    wl = W.fanout("pf-maxq", 54, n_agents=2, prefix=64, suffix_lo=1, suffix_hi=10, hq=32, hkv=8, r=16, chunk=100)
    lw = LoadedWorkload(wl, rope=False)
    st = lw.prefill_setup()
    st["args"].max_q_per_agent = 10          # one block of 64 tokens per agent (4 query heads per KV head)
    st["out"].zero_()
    out = lw.prefill().clone()
    torch.cuda.synchronize()
    o = out.float().cpu().numpy()
    rows = st["rows"]
    for i, a in enumerate(st["agents"]):
        mine = o[i * 100:(i + 1) * 100]
        assert np.isfinite(mine[:64]).all() and np.isnan(mine[64:]).all()
    p = W.oracle_inputs(wl, agents=st["agents"], q_rows={a: np.arange(64) for a in st["agents"]}, rope=False)
    ref = oracle.residual_attention(p)
    pos = {int(x): i for i, x in enumerate(rows)}
    check_close("maxq covered rows", out[[pos[int(x)] for x in p["q_index"]]], ref)
    lw.close()


@pytest.mark.parametrize("r,rope", [(0, False), (8, True), (16, False), (16, True), (32, False), (32, True), (64, False)])
@pytest.mark.parametrize("n_agents", [3, 17])
def test_prefill_row_block_sizes(r, rope, n_agents):
    """Grids that fill at most half of the compute units run 128 query rows per workgroup, larger
    ones 256 (17 agents x 8 KV heads): sequences ending around 64-key tile edges, chunks around
    both row-block sizes (32 and 64 tokens of four heads), one agent without adapter."""
    chunk = [1, 31, 32, 33, 63, 64, 65, 5, 100, 2, 16, 17, 48, 64, 1, 7, 3][:n_agents]
    end = [64, 65, 127, 128, 129, 191, 192, 193, 200, 63, 64, 128, 130, 320, 257, 256, 66][:n_agents]
    suffix = [e - 24 - c if e - 24 - c > 0 else 1 for e, c in zip(end, chunk)]
    wl = W._build("pf-blocks", 77, 32, 8, 128, r, 16, [-1], [24], [0] * n_agents, suffix, chunk, {1} if r else set(), 0.05)
    lw, g, ref = run_prefill(f"row-blocks r={r} rope={rope} agents={n_agents}", wl, rope)
    lw.close()


@pytest.mark.parametrize("r,rope", [(0, False), (8, False), (16, True), (32, False), (32, True), (64, False), (64, True)])
@pytest.mark.parametrize("n_agents", [3, 17])
def test_prefill_row_sums_of_peaked_rows(r, rope, n_agents):
    """Peaked rows (queries of standard deviation 6): the denominator must carry the same bf16
    rounding of the weights as the value products, or a whole row is off by one factor of up to
    1 +- 2^-9.  A dim's values differ little over the keys (1 <= |mean| < 2, deviation 0.05), so the
    weights' rounding itself hardly shows, and the mean relative error of a row's 128 dims is that
    factor plus the mean of 128 roundings of the output to bf16, each at most 2^-8 of the value and
    uniform: standard deviation 2^-8 / sqrt(3 * 128) = 2.0e-4 at most.  One agent has no adapter."""
    rng = np.random.default_rng(3)
    chunk, suffix = [int(c) for c in rng.integers(20, 64, n_agents)], [int(c) for c in rng.integers(5, 300, n_agents)]
    wl = W._build("pf-peaked", 91, 32, 8, 128, r, 16, [-1], [300], [0] * n_agents, suffix, chunk, {1} if r else set(),
                  0.002, q_std=6.0)
    mean = (1 + rng.random((1, 8, 128))) * rng.choice([-1.0, 1.0], (1, 8, 128))
    wl.base_v[:] = W.f32_to_bf16_bits(mean + 0.05 * rng.standard_normal(wl.base_v.shape))
    lw, g, ref = run_prefill(f"peaked r={r} rope={rope} agents={n_agents}", wl, rope)
    lw.close()
    factor = ((g - ref) / ref).mean(axis=-1)
    rms = float(np.sqrt((factor ** 2).mean()))
    print(f"row factor: rms {rms:.3e} max {np.abs(factor).max():.3e}", flush=True)
    assert rms <= 2.0 ** -8 / np.sqrt(3 * 128)


@pytest.mark.parametrize("r,rope", [(8, False), (8, True), (16, False), (16, True), (32, False), (32, True), (64, False), (64, True)])
@pytest.mark.parametrize("hq,hkv,n_agents", [(32, 8, 3), (16, 2, 3), (32, 8, 17)])
def test_prefill_amplified_adapters(r, rope, hq, hkv, n_agents):
    """C B ~ N(0, 1): the value residual acc_r . B_V that the end of the kernel adds is as large as the
    base values, on grids of both row-block sizes and with four and eight query heads per KV head.  The
    context is long enough that no output reaches 4, from where on rounding it to bf16 alone takes 2^-6
    of the bar's 2e-2."""
    wl = W.fanout(f"pf-amp-r{r}", 95, n_agents=n_agents, prefix=600, suffix_lo=1, suffix_hi=60, hq=hq, hkv=hkv, r=r,
                  chunk=45, b_std=1.0 / np.sqrt(r))
    lw, g, ref = run_prefill(f"prefill amplified r={r} rope={rope} hq={hq} hkv={hkv} agents={n_agents}", wl, rope)
    lw.close()


def _block_rows(wl, rope):
    return N.fkv_prefill_block_rows(wl.hq, wl.hkv, wl.r, int(rope), wl.n_agents, max(len(c) for c in wl.chunk_tokens), None)


@pytest.mark.parametrize("r,rope", [(0, False), (8, False), (8, True), (16, False), (16, True), (32, False), (32, True), (64, False)])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (16, 2)])
def test_prefill_long_contexts_in_blocks_of_128_rows(r, rope, hq, hkv):
    """The page ids of 64 tiles at a time and their delay line, whose length depends on rank and RoPE,
    roll over: sequences that end on both sides of tiles 64 and 128.  Residuals as large as the base
    rows, so that a tile's page taken from the wrong place moves the output by a tenth (rel-L2)."""
    end, chunk = [4095, 4097, 4161, 8192, 8200, 8257], [3, 33, 20, 1, 40, 7]
    wl = W._build("pf-long", 96, hq, hkv, 128, r, 16, [-1], [3900], [0] * 6, [e - c - 3900 for e, c in zip(end, chunk)], chunk,
                  {1} if r else set(), 1.0 / np.sqrt(max(r, 1)))
    assert _block_rows(wl, rope) == 128
    lw, g, ref = run_prefill(f"long r={r} rope={rope} hq={hq}", wl, rope, q_sample=lambda n: sorted({0, n // 2, n - 1}))
    lw.close()


@pytest.mark.parametrize("r,rope", [(0, False), (8, False), (8, True), (16, False), (16, True), (32, False)])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (16, 2)])
def test_prefill_long_contexts_in_blocks_of_256_rows(r, rope, hq, hkv):
    """The same on grids that take 256 rows per workgroup: chunks of seventeen blocks and more that begin
    below tile 64 and end behind it, with four and eight query heads per KV head."""
    n = 17 * 256 // (hq // hkv)
    chunk = [n + 9, n // 3, n - 50]
    wl = W._build("pf-long-256", 97, hq, hkv, 128, r, 16, [-1], [3700], [0] * 3, [100, 400, 7], chunk, {1} if r else set(),
                  1.0 / np.sqrt(max(r, 1)))
    assert _block_rows(wl, rope) == 256
    sample = lambda m: sorted({0, 31, 32, 63, 64, m // 2, 4096 - 3800, 4097 - 3800, m - 65, m - 2, m - 1} & set(range(m)))
    lw, g, ref = run_prefill(f"long-256 r={r} rope={rope} hq={hq}", wl, rope, q_sample=sample)
    lw.close()
