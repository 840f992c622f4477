"""GPU parity: the HIP path through the C ABI against the fp64 CPU oracle.

Each case prints its name before touching the GPU.  The comparison bar is
stated in tests/parity.py.
"""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import starkv_oracle as O  # noqa: E402
from paper_2606_01790_amd import starkv as sk  # noqa: E402
from paper_2606_01790_amd import workload as WL  # noqa: E402
from paper_2606_01790_amd.pipeline import ArrayCase, TrajectoryRunner  # noqa: E402
from parity import check_layer, oracle_params  # noqa: E402

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[parity] {msg}", flush=True)


def params_for(cid, prior_active=False):
    p = sk.params_default()
    if cid >= 3:                    # multi-step (AgentNetBench-style) T range
        p.t_min, p.t_max = 0.95, 1.05
    if prior_active:                # lambda_eff = lambda from the first step
        p.n_warmup, p.n_ramp = 0, 0
    return p


class HostFrames:
    """Host copies of a trajectory's inputs, straight from the generator."""

    def __init__(self, spec):
        self.spec = spec
        self.tr = WL.Trajectory(spec)
        self.frames = {}

    def cache(self, layer, step):
        ks, vs = [], []
        for f in self.spec.frames(step):
            if (layer, f) not in self.frames:
                self.frames[(layer, f)] = self.tr.frame_kv(layer, f)
            k, v = self.frames[(layer, f)]
            ks.append(k)
            vs.append(v)
        k, v = self.tr.text_kv(layer, step)
        return np.concatenate(ks + [k], axis=1), np.concatenate(vs + [v], axis=1)


def run_trajectory(cid, layers=None, prior_active=False, steps=None, groups=1,
                   per_head=False, on_step=None, tem_decay="exp", aeb_mode="entropy"):
    """per_head: a subspace per query head; the oracle then scores the cache
    with every shared K group replicated across its heads."""
    spec = WL.SPECS[cid]
    p = params_for(cid, prior_active)
    p.tem_decay, p.aeb_mode = sk.TEM_DECAY[tem_decay], sk.AEB_MODE[aeb_mode]
    op = oracle_params(p)
    say(f"cfg{cid} prior_active={prior_active} per_head={per_head} tem={tem_decay} "
        f"aeb={aeb_mode}: allocate")
    runner = TrajectoryRunner(spec, p, per_head=per_head)
    runner.reset()
    host = HostFrames(spec)
    layers = list(range(spec.n_layers)) if layers is None else list(layers)
    Ns = spec.H if per_head else spec.G
    states = {l: O.LayerState(Ns) for l in layers}
    report = {}
    for step in range(1, (steps or spec.steps) + 1):
        say(f"cfg{cid} step {step}: load + score/update")
        runner.load_step(step)
        if groups > 1:              # the bench's launch: layer groups on streams
            assert len(spec.budgets(step)) == 1
            runner.run_step(step, spec.budgets(step)[0], groups=groups)
        else:
            runner.score_and_update(step)
        L, W = spec.L(step), spec.W
        spans = spec.spans(step)
        budgets = spec.budgets(step)
        orc_base = {}
        for layer in layers:
            K, V = host.cache(layer, step)
            Q = host.tr.window_q(layer, step)
            Ks = WL.to_float64(K, spec.dtype)
            if per_head:
                Ks = O.per_head_cache(Ks, spec.H)
            out, states[layer] = O.compress_layer(
                WL.to_float64(Q, spec.dtype), Ks, None, L, W,
                spans, step, budgets[0], op, states[layer], copy_rows=(K, V))
            orc_base[layer] = (out, K, V)
        for B in budgets:
            say(f"cfg{cid} step {step} B={B}: select/compact")
            if groups <= 1:
                runner.select_and_compact(step, B)
            torch.cuda.synchronize()
            gpu = runner.outputs(step, B)
            for layer in layers:
                out, K, V = orc_base[layer]
                orc = dict(out)
                orc["I"] = O.topb_select(out["s"], B)
                orc["K_out"], orc["V_out"] = O.gather_compact(K, V, orc["I"], L, W)
                g = {k: v[layer] for k, v in gpu.items()}
                check_layer(f"cfg{cid} step{step} L{layer} B{B}", K, V, L, W, spans,
                            step, B, op, Ns, g, orc, report)
        if on_step is not None:
            on_step(step, runner.outputs(step, budgets[-1]), states)
    say(f"cfg{cid} done: max S rel {max(report['S']):.2e}, max s rel "
        f"{max(report['s']):.2e}, idx band tokens {sum(report['idx_band'])}, "
        f"g* near-ties {sum(report['gstar_ties'])}")
    return report


def test_config1_tiny_f32():
    run_trajectory(1)


def test_config2_single_layer_bf16():
    run_trajectory(2)


def test_config2_prior_active():
    run_trajectory(2, prior_active=True)


def test_config3_28_layers_5_steps():
    run_trajectory(3)


def test_config3_prior_active_sampled_layers():
    run_trajectory(3, layers=[0, 1, 2, 3, 27], prior_active=True)


def test_config3_layer_groups_on_two_streams():
    """The bench's launch configuration: each step as two layer groups on two
    HIP streams (the second group's scoring overlaps the first group's
    statistics, selection and gather); layers at both group edges."""
    run_trajectory(3, layers=[0, 13, 14, 27], prior_active=True, groups=2)


def test_config4_budget_sweep_sampled_layers():
    """15 steps, three budgets per step; the oracle follows layers 0, 9, 18
    and 27 through the whole trajectory (their state depends on every
    step)."""
    run_trajectory(4, layers=[0, 9, 18, 27])


def oracle_state_from_gpu(state_bytes_np, layer, G, frame_cap):
    """The oracle's LayerState equal to one layer's GPU state block: a 64-byte
    header (int32 magic, G, frame_cap, n, nf, ...), MI_bar[G] float32 padded
    to 16 bytes, then m[G][frame_cap] float32; blocks padded to 256 bytes."""
    m_off = 64 + (G * 4 + 15) // 16 * 16
    stride = (m_off + G * frame_cap * 4 + 255) // 256 * 256
    blk = state_bytes_np[layer * stride:(layer + 1) * stride]
    hdr = blk[:64].view(np.int32)
    n, nf = int(hdr[3]), int(hdr[4])
    mi_bar = blk[64:64 + 4 * G].view(np.float32).astype(np.float64)
    m = blk[m_off:m_off + 4 * G * frame_cap].view(np.float32).reshape(G, frame_cap)
    return O.LayerState(G, mi_bar, m[:, :nf].astype(np.float64), n)


def test_config5_long_trajectory_sampled_steps():
    """The 30-step 2560x1440 trajectory (W = 64: 448 window rows per group,
    up to 140K past tokens, keys beyond every LDS cache) for layers 0 and 27
    on the GPU.  Layer 0: the oracle carries its own state through all 30
    steps; at steps 1, 2, 16 and 30 every output is compared, and so are the
    stability means m_g and MI_bar the GPU state holds afterwards (the
    stability row of 4641 tokens, sec. 3.5).  Layer 27: at the same steps the
    oracle runs that step from the GPU's own state after the previous one."""
    spec = WL.SPECS[5]
    p = params_for(5)
    op = oracle_params(p)
    layers = [0, 27]
    host = HostFrames(spec)
    frame_cap = spec.n_frame
    case = ArrayCase(spec.H, spec.G, spec.d, spec.W, len(layers), spec.L(spec.steps),
                     spec.dtype, p, frame_cap)
    own = O.LayerState(spec.G)          # layer 0's oracle state, every step
    report = {}
    for step in range(1, spec.steps + 1):
        L, spans, B = spec.L(step), spec.spans(step), spec.budgets(step)[0]
        caches = [host.cache(layer, step) for layer in layers]
        Ks = np.stack([c[0] for c in caches])
        Vs = np.stack([c[1] for c in caches])
        Qs = np.stack([host.tr.window_q(layer, step) for layer in layers])
        check = step in (1, 2, 16, 30)
        prev = case.state.cpu().numpy()
        say(f"cfg5 step {step}: L={L} B={B}{' (checked)' if check else ''}")
        gpu = case.run(Qs, Ks, Vs, L, spans, step, B)
        out0, own = O.compress_layer(WL.to_float64(Qs[0], spec.dtype),
                                     WL.to_float64(Ks[0], spec.dtype), None, L, spec.W,
                                     spans, step, B, op, own, copy_rows=(Ks[0], Vs[0]))
        if not check:
            continue
        after = case.state.cpu().numpy()
        for i, layer in enumerate(layers):
            if i == 0:
                out = out0
            else:
                st = oracle_state_from_gpu(prev, i, spec.G, frame_cap)
                out, _ = O.compress_layer(WL.to_float64(Qs[i], spec.dtype),
                                          WL.to_float64(Ks[i], spec.dtype), None, L, spec.W,
                                          spans, step, B, op, st, copy_rows=(Ks[i], Vs[i]))
            g = {k: v[i] for k, v in gpu.items()}
            check_layer(f"cfg5 step{step} L{layer}", Ks[i], Vs[i], L, spec.W, spans, step,
                        B, op, spec.G, g, out, report)
        gst = oracle_state_from_gpu(after, 0, spec.G, frame_cap)
        assert gst.n == own.n == step
        assert gst.m.shape == own.m.shape == (spec.G, spec.n_frame)
        np.testing.assert_allclose(gst.m, own.m, rtol=1e-3, atol=1e-9,
                                   err_msg=f"cfg5 step{step}: stability means m_g")
        assert np.max(np.abs(gst.mi_bar - own.mi_bar)) <= 2e-3, f"cfg5 step{step}: MI_bar state"
    say(f"cfg5 done: max S rel {max(report['S']):.2e}, idx band tokens "
        f"{sum(report['idx_band'])}, rank-bin near-tie moves {sum(report['bin_moves'])}")


def test_determinism_bitwise():
    spec = WL.SPECS[2]
    p = params_for(2, prior_active=True)
    outs = []
    for rep in range(2):
        say(f"determinism run {rep}")
        r = TrajectoryRunner(spec, p)
        r.reset()
        r.load_step(1)
        r.run_step(1, spec.budgets(1)[0])
        torch.cuda.synchronize()
        outs.append(r.outputs(1, spec.budgets(1)[0]))
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("fused", [False, True])
def test_graph_replay_matches_eager(fused):
    """A trajectory step (fresh state, four calls, or three with the
    statistics and the selection in one call) captured into a HIP graph:
    every replay, with eager work between replays, reproduces the eager run
    of the four separate calls bit for bit."""
    spec = WL.SPECS[3]
    p = params_for(3, prior_active=True)
    r = TrajectoryRunner(spec, p)
    for s in (1, 2):
        r.load_step(s)     # caches hold step 2's text; step 1 only reads frame 1 + text
    # eager reference: the separate calls on the same buffers as the graph
    def traj(fused_calls):
        sk.state_init(r.dims(spec.peak_step), r.state, r.frame_cap)
        r.run_step(2, spec.budgets(2)[0], fused=fused_calls)
    say(f"graph (fused {fused}): eager reference")
    traj(False)
    torch.cuda.synchronize()
    ref = r.outputs(2, spec.budgets(2)[0])
    g = torch.cuda.CUDAGraph()
    say("graph: capture")
    with torch.cuda.graph(g):
        traj(fused)
    for rep in range(3):
        r.S.zero_()
        r.s.zero_()
        r.idx.zero_()
        r.k_out.zero_()
        torch.cuda.synchronize()
        say(f"graph: replay {rep}")
        g.replay()
        torch.cuda.synchronize()
        out = r.outputs(2, spec.budgets(2)[0])
        for k in ref:
            assert np.array_equal(ref[k], out[k]), (rep, k)
        traj(fused)                  # eager work between replays
        torch.cuda.synchronize()


# ------------------------------------------------------------------ edge cases

def run_case(tag, H, G, d, W, L, spans, F, B, dtype, p, seed=0, n_layers=2,
             L_cap=None, Qs=None, Ks=None, Vs=None, case=None, states=None,
             per_head=False):
    L_cap = L_cap or L
    if Qs is None:
        Qs, Ks, Vs = WL.random_case(seed, n_layers, H, G, d, L_cap, W, dtype)
    frame_cap = max([r * c for (_, r, c, _) in spans] + [1])
    case = case or ArrayCase(H, G, d, W, n_layers, L_cap, dtype, p, frame_cap,
                             per_head=per_head)
    say(f"{tag}: H={H} G={G} d={d} W={W} L={L} B={B} {dtype} per_head={per_head}")
    gpu = case.run(Qs, Ks, Vs, L, spans, F, B)
    op = oracle_params(p)
    Ns = H if per_head else G
    states = states if states is not None else [O.LayerState(Ns) for _ in range(n_layers)]
    report = {}
    for layer in range(n_layers):
        K = Ks[layer][:, :L]
        V = Vs[layer][:, :L]
        Kq = WL.to_float64(K, dtype)
        if per_head:
            Kq = O.per_head_cache(Kq, H)
        out, states[layer] = O.compress_layer(
            WL.to_float64(Qs[layer], dtype), Kq, None, L, W, spans,
            F, B, op, states[layer], copy_rows=(K, V))
        g = {k: v[layer] for k, v in gpu.items()}
        check_layer(f"{tag} L{layer}", K, V, L, W, spans, F, B, op, Ns, g, out, report)
    return case, states


def test_ragged_rows_and_tokens_bf16():
    """R = 5*7 = 35 window rows (a padded MFMA block), L_p = 1000 (a ragged
    token tail), spans at odd offsets with text between them."""
    p = params_for(3, prior_active=True)
    spans = [(3, 7, 11, 1), (100, 13, 9, 2), (300, 20, 30, 3)]
    run_case("ragged", 28, 4, 128, 5, 1005, spans, 3, 137, "bf16", p, seed=1)


@pytest.mark.parametrize("Lp", [1, 31, 33, 257, 260, 288, 292, 319, 511, 513, 1100])
def test_token_tail_sweep(Lp):
    """Past-token counts around the 32-token MFMA blocks and the 256-token
    chunks: waves and lane halves that see only masked tokens."""
    p = params_for(2)
    W = 8
    L = Lp + W
    n = min(Lp, 12) * min(max(Lp // 12, 1), 10)
    spans = [(0, min(Lp, 12), min(max(Lp // 12, 1), 10), 1)] if n <= Lp else []
    run_case(f"tail Lp={Lp}", 8, 2, 64, W, L, spans, 1, max(Lp // 5, 1), "bf16", p,
             seed=Lp)


@pytest.mark.parametrize("nrb,per_head", [(n, False) for n in range(1, 15)]
                         + [(n, True) for n in range(2, 15)])
def test_slab_row_block_sweep(nrb, per_head):
    """Every row-block count at a call of few slabs, whose pass 2 (and pass 1,
    but for 9 to 11 row blocks) is the small-call kernel (bf16, d = 128): with a subspace per group, W = 32*nrb - 8 rows of one head (a padded last
    row block); with a subspace per head, nrb >= 2 heads of W = 32 rows (one
    row block each, one output per stage; one head per group is the
    per-group case).  L_p = 300: four full 64-token slabs
    and a ragged one."""
    p = params_for(2, prior_active=True)
    G = 2
    H, W = (G * nrb, 32) if per_head else (G, 32 * nrb - 8)
    Lp = 300
    spans = [(4, 12, 20, 1)]
    run_case(f"slab nrb={nrb} per_head={per_head}", H, G, 128, W, Lp + W, spans, 1, 50,
             "bf16", p, seed=100 + nrb, n_layers=1, per_head=per_head)


@pytest.mark.parametrize("k,Lp", [(1, 1), (3, 5), (5, 255), (7, 257), (9, 1025), (63, 700)])
def test_pool_width_sweep(k, Lp):
    """AvgPool1D widths from 1 to 63 (the widest accepted), with token counts
    on both sides of the pooling kernel's 256-token tiles and a pool wider
    than a short row (zero padding on both sides, halos crossing tiles)."""
    p = params_for(2)
    p.pool_kernel = k
    W = 8
    L = Lp + W
    rows, cols = min(Lp, 10), max(min(Lp // 10, 12), 1)
    spans = [(0, rows, cols, 1)] if rows * cols <= Lp else []
    run_case(f"pool k={k} Lp={Lp}", 8, 2, 64, W, L, spans, 1, max(Lp // 5, 1), "bf16", p,
             seed=40 + k)


def test_budget_extremes():
    p = params_for(2)
    spans = [(0, 10, 20, 1)]
    for B in (0, 1, 400 - 8):
        run_case(f"B={B}", 8, 2, 64, 8, 400, spans, 1, B, "bf16", p, seed=2)


def test_mha_f32_d128_and_strided_cache():
    """G = H (per-head subspaces) in fp32 with d = 128, cache capacity above L."""
    p = params_for(2)
    spans = [(0, 12, 16, 1)]
    run_case("mha", 4, 4, 128, 4, 250, spans, 1, 40, "f32", p, seed=3, L_cap=333)


def test_exact_ties_everywhere():
    """All keys zero: uniform attention, so scores tie exactly in the interior.
    Rank bins and the top-B cut must then follow token order on both sides."""
    p = params_for(2, prior_active=True)
    H, G, d, W, L = 8, 2, 128, 8, 600
    Qs, Ks, Vs = WL.random_case(4, 2, H, G, d, L, W, "bf16")
    Ks = np.zeros_like(Ks)
    spans = [(10, 20, 25, 1)]
    run_case("ties", H, G, d, W, L, spans, 1, 50, "bf16", p, Qs=Qs, Ks=Ks, Vs=Vs)


@pytest.mark.parametrize("dtype,d,H,G,W", [("bf16", 128, 28, 4, 32), ("f32", 64, 16, 2, 16)])
def test_rising_and_spiking_logits(dtype, d, H, G, W):
    """Pass 1 keeps a row's reference logit until a block's sum would leave
    [0, 2^32).  Layer 0: keys scaled up along the token index, so the logits
    of most rows keep rising within every chunk.  Layer 1: spike keys equal
    to s times one window query (s = 2, 4, 12), whose logit for that row sits
    about 30, 65 and 200 log2 units above the rest: the last overflows the
    block sum to +inf.  Spikes fall in the first block, mid-chunk, on a tile
    edge and on the last past token."""
    p = params_for(2, prior_active=True)
    L = 3000 + W
    Lp = L - W
    Qs, Ks, Vs = WL.random_case(12, 2, H, G, d, L, W, dtype)
    Qf = WL.to_float64(Qs, dtype).astype(np.float32)
    Kf = WL.to_float64(Ks, dtype).astype(np.float32)
    ramp = (1.0 + 3.0 * np.arange(L, dtype=np.float32) / L)[:, None]
    Kf[0] *= ramp[None]
    hpg = H // G
    for i, (t, s) in enumerate([(5, 12.0), (300, 2.0), (767, 4.0), (1024, 12.0),
                                (1535, 2.0), (2000, 4.0), (Lp - 1, 12.0)]):
        for g in range(G):
            h = g * hpg + (i + g) % hpg
            Kf[1, g, t] = s * Qf[1, h, (t + g) % W]
    if dtype == "bf16":
        Ks = WL.f32_to_bf16_bits(Kf)
    else:
        Ks = Kf
    spans = [(0, 40, 60, 1), (2400, 20, 30, 2)]
    run_case(f"rising {dtype}", H, G, d, W, L, spans, 2, 400, dtype, p, Qs=Qs, Ks=Ks,
             Vs=Vs)


@pytest.mark.parametrize("kind", ["zero", "three"])
def test_ties_beyond_the_key_cache(kind):
    """30,000 visual tokens, more than the statistics kernel keeps in LDS, so
    every rank-binning pass reads S from memory.  Keys all zero (every
    interior score ties) or drawn from three one-hot vectors (three values,
    each shared by about 10,000 tokens): the bin edges fall inside runs of equal
    keys, split by token order.  The three-vector case pools over one token:
    a wider pool mixes neighbours, and neighbourhoods that are permutations
    of each other give equal sums that float32 and float64 round apart, so
    the two sides would order those tokens differently."""
    p = params_for(2, prior_active=True)
    if kind == "three":
        p.pool_kernel = 1
    H, G, d, W, L = 8, 2, 128, 8, 30100
    Qs, Ks, Vs = WL.random_case(5, 1, H, G, d, L, W, "bf16")
    if kind == "zero":
        Ks = np.zeros_like(Ks)
    else:
        # zero, 2 e_3 or -e_7: every logit is one exact product, so equal keys
        # give bit-equal scores on both sides whatever the summation order
        basis = np.zeros((3, d), np.float32)
        basis[1, 3], basis[2, 7] = 2.0, -1.0
        pick = np.random.default_rng([5, 3]).integers(0, 3, size=(1, G, L))
        Ks = WL.f32_to_bf16_bits(basis[pick])
    spans = [(10, 150, 200, 1)]
    run_case(f"ties uncached {kind}", H, G, d, W, L, spans, 1, 3000, "bf16", p, Qs=Qs,
             Ks=Ks, Vs=Vs, n_layers=1)


@pytest.mark.parametrize("rows,cols", [(50, 60), (150, 200)])
def test_pairwise_tied_keys(rows, cols):
    """Every odd token repeats the key of the token before it, and the pool
    covers one token, so scores tie in pairs and bin edges fall inside ties.
    3,000 visual tokens keep their keys in LDS; 30,000 do not.  Both take the
    fused binning pass, which splits a tie at an edge by token order among
    the kept keys."""
    p = params_for(2, prior_active=True)
    p.pool_kernel = 1
    H, G, d, W = 8, 2, 128, 8
    L = rows * cols + 100
    Qs, Ks, Vs = WL.random_case(9, 1, H, G, d, L, W, "bf16")
    Ks = Ks.copy()
    Ks[:, :, 1::2] = Ks[:, :, 0:-1:2][:, :, :Ks[:, :, 1::2].shape[2]]
    spans = [(10, rows, cols, 1)]
    run_case(f"pair ties {rows}x{cols}", H, G, d, W, L, spans, 1, rows * cols // 5, "bf16", p,
             Qs=Qs, Ks=Ks, Vs=Vs, n_layers=1)


@pytest.mark.parametrize("scale", [1, 10])
def test_sixty_four_spans_of_odd_shapes(scale):
    """The maximum of 64 visual spans (one frame each, three text tokens
    between them), cycling through 1x1, one row of 150*scale, one column of
    150*scale, 7x9, 13x17, 3x(10*scale), (4*scale)x(4*scale) and 2x3: rows
    longer than the 1024-token step of a pass, one-column spans, and many
    span changes per thread.  About 5,200 visual tokens at scale 1 (keys
    kept in LDS) and 41,500 at scale 10 (keys read from memory)."""
    p = params_for(3, prior_active=True)
    shapes = [(1, 1), (1, 150 * scale), (150 * scale, 1), (7, 9), (13, 17), (3, 10 * scale),
              (4 * scale, 4 * scale), (2, 3)]
    spans, t = [], 5
    for f in range(64):
        r, c = shapes[f % len(shapes)]
        spans.append((t, r, c, f + 1))
        t += r * c + 3
    H, G, d, W = 8, 2, 64, 8
    L = t + 40 + W
    n_vis = sum(r * c for _, r, c, _ in spans)
    run_case(f"64 spans x{scale}", H, G, d, W, L, spans, 64, n_vis // 10, "bf16", p, seed=17,
             n_layers=1)


@pytest.mark.parametrize("n_bins,grid", [(1, 8), (2, 1), (8, 16), (16, 8), (33, 4), (64, 16)])
@pytest.mark.parametrize("rows,cols", [(40, 60), (150, 160)])
def test_rank_bins_and_grid_extremes(n_bins, grid, rows, cols):
    """Rank-bin counts K from 1 (no edges) to 64 and grids M from 1 to 16,
    with 2,400 visual tokens (keys in LDS) and 24,000 (keys read from
    memory): K = 33 is the largest that takes the fused pass, K = 64 with
    M = 16 fills the whole joint histogram.  MI and w are compared stage-wise
    and end to end, with the prior active (lambda = 0.5 from the first
    step).  On random inputs the two groups' MIs can lie within rounding of
    each other (1.5e-4 apart at K = 33 on 24,000 tokens), where min-max
    ranks them either way: the near-tie rule of tests/parity.py then takes
    the oracle's fusion with the GPU's w."""
    p = params_for(2, prior_active=True)
    p.n_bins, p.grid = n_bins, grid
    H, G, d, W = 8, 2, 64, 8
    L = rows * cols + 200
    spans = [(100, rows, cols, 1)]
    run_case(f"K={n_bins} M={grid} {rows}x{cols}", H, G, d, W, L, spans, 1, rows * cols // 4,
             "bf16", p, seed=n_bins * 31 + grid, n_layers=1)


def test_frame_size_change_resets_stability():
    """Two steps whose current frames differ in size: m_g restarts, phi = 0."""
    p = params_for(3, prior_active=True)
    H, G, d, W = 8, 2, 64, 8
    L1, L2 = 300, 500
    case = None
    states = None
    seq = [(L1, [(0, 10, 20, 1)], 1),
           (L2, [(0, 10, 20, 1), (250, 12, 15, 2)], 2),
           (L2, [(0, 10, 20, 1), (250, 12, 15, 2)], 2)]
    for step, (L, spans, F) in enumerate(seq, 1):
        Qs, Ks, Vs = WL.random_case(10 + step, 2, H, G, d, L, W, "bf16")
        if case is None:
            case = ArrayCase(H, G, d, W, 2, L2, "bf16", p, 200)
        case, states = run_case(f"resize step{step}", H, G, d, W, L, spans, F, 60,
                                "bf16", p, n_layers=2, Qs=Qs, Ks=Ks, Vs=Vs, case=case,
                                states=states)
    assert states[0].m.shape == (2, 180)


# ------------------------------------------------- per-head subspaces (MHA-head)

def test_per_head_config2_shape():
    """Qwen2.5-VL-7B shape (H=28 over G=4 groups, W=32, one 1920x1080 frame):
    28 subspaces, one per head, every pass-2 row block a whole head."""
    spec = WL.SPECS[2]
    p = params_for(2, prior_active=True)
    spans = spec.spans(1)
    run_case("per-head cfg2", spec.H, spec.G, spec.d, spec.W, spec.L(1), spans, 1,
             spec.budgets(1)[0], "bf16", p, seed=31, n_layers=1, per_head=True)


@pytest.mark.parametrize("H,G,W,dtype,d", [(4, 2, 8, "f32", 64), (28, 4, 16, "bf16", 128),
                                           (14, 2, 40, "bf16", 64), (8, 2, 64, "bf16", 128)])
def test_per_head_window_row_layouts(H, G, W, dtype, d):
    """Heads of W = 8, 16 and 40 rows (partials per 8-row group, a head split
    across row blocks at W = 40) and of W = 64 (two whole row blocks)."""
    p = params_for(2, prior_active=True)
    spans = [(5, 12, 15, 1), (200, 12, 15, 2)]
    L = 420 + W
    run_case(f"per-head W={W}", H, G, d, W, L, spans, 2, 97, dtype, p, seed=W,
             per_head=True)


def test_per_head_trajectory_state():
    """Five steps of the 28-layer trajectory with per-head subspaces: the MI
    EMA and the stability means of 28 subspaces carried across steps."""
    run_trajectory(3, layers=[0, 27], prior_active=True, per_head=True)


def test_per_head_flag_is_identity_under_mha():
    """G = H: a subspace per group and per head are the same thing, so both
    settings give bit-identical outputs."""
    p = params_for(2, prior_active=True)
    spans = [(0, 10, 12, 1)]
    outs = []
    for ph in (False, True):
        Qs, Ks, Vs = WL.random_case(41, 2, 4, 4, 64, 300, 8, "bf16")
        case = ArrayCase(4, 4, 64, 8, 2, 300, "bf16", p, 120, per_head=ph)
        say(f"mha per_head={ph}")
        outs.append(case.run(Qs, Ks, Vs, 300, spans, 1, 50))
    for k in outs[0]:
        assert np.array_equal(outs[0][k], outs[1][k]), k


# ------------------------------------- image slots and a resolution change

def test_config6_image_slots_and_resolution_change():
    """Ten steps with image_slots = 5 (frames leave the context from step 6,
    every token after them moves) and the screen switching from 1920x1080 to
    1280x720 at frame 7.  The stability means follow the newest frame, so
    phi is exactly 0 at step 1 and at step 7, where the frame's token count
    changes, and positive in the steps in between and after (S is never
    orthogonal to the previous means here)."""
    spec = WL.SPECS[6]
    G = spec.G

    def on_step(step, gpu, states):
        phi = gpu["scal"][:, 3 * G:4 * G]
        if step in (1, 7):
            assert np.all(phi == 0.0), f"step {step}: phi {phi[:2]}"
        else:
            assert np.all(phi > 0.0), f"step {step}: phi {phi[:2]}"

    run_trajectory(6, layers=[0, 1, 27], prior_active=True, on_step=on_step)


# ------------------------------------------- ablation variants (sec. 4.2)

@pytest.mark.parametrize("tem,aeb", [("linear", "entropy"), ("gamma", "confidence"),
                                     ("exp", "confidence")])
def test_ablation_variants_trajectory(tem, aeb):
    """The linear and gamma temporal decays and the confidence-based AEB on
    the 28-layer trajectory (discount active from step 2, prior active),
    layers 0 and 27, against the oracle with the same readings."""
    run_trajectory(3, layers=[0, 27], prior_active=True, tem_decay=tem, aeb_mode=aeb)


def test_confidence_aeb_single_frame():
    """One 1920x1080 frame with the single-image T range [0.75, 1.25]: the
    temperature comes from the peak base-score mass."""
    run_trajectory(2, prior_active=True, aeb_mode="confidence")


# ------------------------------------------------ largest shapes, no spans

def test_largest_window_row_block_bf16():
    """R = W * H / G = 512 window rows per group (16 MFMA row blocks, the
    largest accepted; d = 64 so that the rows fit the 128 KiB row budget)."""
    p = params_for(2, prior_active=True)
    spans = [(40, 18, 24, 1)]
    run_case("R=512", 32, 2, 64, 32, 900, spans, 1, 120, "bf16", p, seed=61, n_layers=1)


def test_largest_window_row_block_f32():
    """R = 128 window rows in fp32 (four row blocks, the fp32 maximum)."""
    p = params_for(2, prior_active=True)
    spans = [(0, 10, 20, 1)]
    run_case("R=128 f32", 8, 2, 64, 32, 400, spans, 1, 60, "f32", p, seed=62, n_layers=1)


def _bf16_unit_bits(rng, shape):
    """bf16 bit patterns of magnitude in [1, 2) with random sign: random
    64-bit words, each read as four bf16 values whose exponent bits are then
    fixed at 127 (sign and seven mantissa bits stay random)."""
    n = int(np.prod(shape))
    assert n % 4 == 0
    u = rng.integers(0, np.iinfo(np.uint64).max, n // 4, dtype=np.uint64, endpoint=True)
    u &= np.uint64(0x807F807F807F807F)
    u |= np.uint64(0x3F803F803F803F80)
    return u.view(np.uint16).reshape(shape)


def test_maximum_size_sixteen_million_visual_tokens():
    """One 4000 x 4000 frame (N = 16e6 visual tokens, just under the 2^24
    limit of the fused rank/joint-histogram path) in a cache of two KV groups
    at d = 128: group 1's rows run from 2.05e9 to 4.1e9 elements into the K
    cache, past 2^31 elements and 2^32 bytes (64-bit offsets in scoring and
    in the gather), the rank pass runs uncached at its
    largest and the selection streams 16e6 far keys.  Group 0's keys in the
    lower half of the frame have half the magnitude, so its scores carry
    spatial structure and its MI stands far above group 1's estimator bias
    (the min-max prior is then well conditioned end to end)."""
    p = params_for(3, prior_active=True)
    rows = cols = 4000
    N = rows * cols
    H, G, d, W = 4, 2, 128, 8
    L = 500 + N + 500 + W
    B = N // 100
    r = np.random.default_rng([64, 1])
    Qs = WL.f32_to_bf16_bits(r.standard_normal((1, H, W, d), dtype=np.float32) *
                             np.float32(0.3))
    Ks = _bf16_unit_bits(r, (1, G, L, d))
    Vs = _bf16_unit_bits(r, (1, G, L, d))
    Ks[0, 0, 500 + N // 2:500 + N] &= np.uint16(0xFF7F)   # exponent 127 -> 126
    assert G * L * d > 2 ** 31 and G * L * d * 2 > 2 ** 32
    say(f"max size: inputs generated, K {Ks.nbytes / 2 ** 30:.1f} GiB")
    run_case("max size", H, G, d, W, L, [(500, rows, cols, 1)], 1, B, "bf16", p,
             n_layers=1, Qs=Qs, Ks=Ks, Vs=Vs)


def test_no_visual_spans():
    """A text-only cache: no visual token, so MI = 0 and phi = 0 in every
    group, D = 1, and the selection runs on s-bar alone."""
    p = params_for(2, prior_active=True)
    _, states = run_case("no spans", 8, 2, 64, 8, 500, [], 0, 80, "bf16", p, seed=63)
    for st in states:
        assert np.all(st.mi_bar == 0.0)


def _random_configuration(seed):
    """A seeded draw over the ABI's shapes and parameters: dtype, head size,
    groups and heads per group, window, subspace granularity, frames with
    text between them, budget, bins, grid, pooling width, the decay and AEB
    variants and whether the prior is active.  Shapes the ABI rejects are
    redrawn."""
    rng = np.random.default_rng(7000 + seed)
    while True:
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        d = int(rng.choice([64, 128]))
        G = int(rng.choice([1, 2, 4, 8]))
        hpg = int(rng.choice([1, 2, 4, 7]))
        W = int(rng.choice([8, 16, 24, 32, 40]))
        per_head = bool(rng.random() < 0.3)
        H = G * hpg
        Rpad = (W * hpg + 31) // 32 * 32
        esz = 4 if dtype == "f32" else 2
        if Rpad > (128 if dtype == "f32" else 512) or Rpad * (d * esz + 16) > 128 * 1024:
            continue
        break
    spans, t = [], int(rng.integers(0, 40))
    for f in range(1, int(rng.integers(1, 5)) + 1):
        rows, cols = int(rng.integers(2, 30)), int(rng.integers(2, 40))
        spans.append((t, rows, cols, f))
        t += rows * cols + int(rng.integers(0, 60))
    Lp = t + int(rng.integers(1, 50))
    p = sk.params_default()
    p.n_bins = int(rng.integers(1, 21))
    p.grid = int(rng.integers(1, 13))
    p.pool_kernel = int(rng.choice([1, 3, 5, 7, 9, 15]))
    p.tem_decay = sk.TEM_DECAY[str(rng.choice(list(sk.TEM_DECAY)))]
    p.aeb_mode = sk.AEB_MODE[str(rng.choice(list(sk.AEB_MODE)))]
    if rng.random() < 0.5:
        p.n_warmup, p.n_ramp = 0, 0
    B = int(rng.integers(0, Lp + 1))
    return dict(H=H, G=G, d=d, W=W, L=Lp + W, spans=spans, F=len(spans), B=B,
                dtype=dtype, p=p, per_head=per_head)


@pytest.mark.parametrize("seed", range(48))
def test_random_configurations(seed):
    """Forty-eight seeded configurations drawn over shapes and parameters, each
    compared with the oracle on two layers at the same bar as the targeted
    cases."""
    c = _random_configuration(seed)
    run_case(f"random {seed}", c["H"], c["G"], c["d"], c["W"], c["L"], c["spans"], c["F"],
             c["B"], c["dtype"], c["p"], seed=seed, per_head=c["per_head"])


@pytest.mark.parametrize("seed", range(12))
def test_random_trajectories(seed):
    """Twelve seeded three-step trajectories: a random configuration whose
    frames arrive one per step (sizes may differ from frame to frame), the
    layer state carried on the GPU and in the oracle, every step compared."""
    c = _random_configuration(100 + seed)
    rng = np.random.default_rng(9000 + seed)
    spans, t = [], int(rng.integers(0, 40))
    for f in range(1, 4):
        rows, cols = int(rng.integers(2, 30)), int(rng.integers(2, 40))
        spans.append((t, rows, cols, f))
        t += rows * cols + int(rng.integers(0, 60))
    L_cap = t + int(rng.integers(1, 50)) + c["W"]
    frame_cap = max(r * cc for (_, r, cc, _) in spans)
    case = ArrayCase(c["H"], c["G"], c["d"], c["W"], 2, L_cap, c["dtype"], c["p"], frame_cap,
                     per_head=c["per_head"])
    states = None
    for step in range(1, 4):
        cur = spans[:step]
        L = cur[-1][0] + cur[-1][1] * cur[-1][2] + int(rng.integers(1, 30)) + c["W"]
        L = min(L, L_cap)
        B = int(rng.integers(0, L - c["W"] + 1))
        case, states = run_case(f"random trajectory {seed} step {step}", c["H"], c["G"], c["d"],
                                c["W"], L, cur, step, B, c["dtype"], c["p"], seed=seed * 10 + step,
                                L_cap=L_cap, case=case, states=states, per_head=c["per_head"])
