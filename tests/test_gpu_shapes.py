"""GPU parity at the benchmark's shapes: the per-layer launch configuration depends on (batch, heads, head_dim,
context, tier mix), not on the layer count, so these cases keep the full per-layer shape of the benchmark configurations and
cut the number of layers (and, for the production-batch config, the number of sequences) to what the CPU oracle
finishes in seconds.  Every output element and every score is compared, not a sample."""
import dataclasses

import numpy as np
import pytest
import torch

from tkv_synth import CONFIGS, small_config

pytestmark = pytest.mark.gpu


def _run_shape(cfg, mode, steps_before=1, steps_after=2):
    from gpu_common import Pair, assert_out_close, assert_scores_close, to_f64
    print(f"[case] {cfg.name}-shaped L={cfg.n_layers} B={cfg.batch} Hq={cfg.n_q_heads} Hkv={cfg.n_kv_heads} D={cfg.head_dim} "
          f"ctx={cfg.context} t2={cfg.t2_format} mode={mode}", flush=True)
    p = Pair(cfg, prefetch_mode=mode)
    L = cfg.n_layers
    k_all, v_all, q_all = p.wl.decode_inputs(0, steps_before + steps_after)
    calls, worst = 0, 0.0

    def step(s):
        nonlocal calls, worst
        out = p.gpu.decode_step(k_all[s], v_all[s], q_all[s])
        for l in range(L):
            p.orc.append(l, to_f64(k_all[s, l]), to_f64(v_all[s, l]))
            ref = p.orc.attend_and_score(l, to_f64(q_all[s, l]))
            worst = max(worst, assert_out_close(to_f64(out[l]), ref, cfg.kv_dtype, f"step {s} layer {l}"))
            calls += 1

    for s in range(steps_before):
        step(s)
    n = p.gpu.layer_length(0)
    p.gpu.classify(cfg.policy_ppm)
    plan = p.gpu.get_pending_tiers()[:, :n]
    want = p.orc.classify(cfg.policy_ppm, score_f32=p.gpu.get_scores())[:, :n]
    assert np.array_equal(plan, want)
    p.gpu.migrate()
    p.orc.migrate()
    for s in range(steps_before, steps_before + steps_after):
        step(s)
    ss = 1.0 / (cfg.n_layers * cfg.n_q_heads)
    n = p.gpu.layer_length(0)
    assert_scores_close(p.gpu.get_scores(), p.orc.score, n, calls * cfg.n_q_heads * ss)
    st = p.gpu.get_stats()
    print(f"[case] worst output error {worst:.2e} of the head max-norm; tiers {st['tier_count']}", flush=True)
    assert st["tier_count"][1] > 0 and st["tier_count"][2] > 0
    p.close()


def test_14b_shape():
    _run_shape(dataclasses.replace(CONFIGS["14b"], n_layers=2, decode_steps=3), "lazy")


def test_7b_shape():
    _run_shape(dataclasses.replace(CONFIGS["7b"], n_layers=2, decode_steps=3), "wait")


def test_32b_shape():
    _run_shape(dataclasses.replace(CONFIGS["32b"], n_layers=1, decode_steps=3), "lazy")


def test_prod_shape_all_64_sequences_one_workgroup_per_pair():
    """The production-batch launch as the bench runs it: 64 sequences x 4 kv heads = 256 pairs, so every pair gets ONE
    workgroup (S = 1) whose eight waves share all F tiles and all int4 Q tiles of a 16384-token list.  The GPU runs
    the whole batch; four of its sequences (first, last, two in between) are checked against an oracle that holds
    just those four (sequences are independent): outputs, scores after a forced four-tier plan, and a chunk of three
    query tokens through the matrix-core launch at the same shape."""
    import paper_2605_09490_amd as tkv
    from gpu_common import assert_out_close, assert_scores_close, to_f64
    from oracle import tkv_oracle as O
    from tkv_synth import Workload
    cfg = dataclasses.replace(CONFIGS["prod"], n_layers=1, decode_steps=5)
    pick = [0, 21, 42, 63]
    print(f"[case] prod-shaped, all {cfg.batch} sequences, ctx={cfg.context}, checking sequences {pick}", flush=True)
    wl = Workload(cfg, device="cuda")
    gpu = tkv.TieredKV(cfg.n_layers, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens,
                       kv_dtype=cfg.kv_dtype, t2_format=cfg.t2_format, k_sink=cfg.k_sink, k_window=cfg.k_window,
                       prefetch_mode="lazy")
    orc = O.OracleCache(cfg.n_layers, len(pick), cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens,
                        kv_dtype=cfg.kv_dtype, t2_format=cfg.t2_format, k_sink=cfg.k_sink, k_window=cfg.k_window)
    k, v = wl.context_kv(0)
    gpu.append(0, k, v)
    orc.append(0, to_f64(k[pick]), to_f64(v[pick]))
    del k, v
    n = cfg.context
    rng = np.random.default_rng(3)
    tiers = rng.choice(4, size=(cfg.batch, n), p=(0.4, 0.37, 0.2, 0.03)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, n - 128:] = 0
    gpu.set_tiers(tiers); gpu.migrate()
    orc.set_tiers(tiers[pick]); orc.migrate()
    calls = 0
    for step in range(2):
        ks, vs = wl.step_kv(step, 0)
        q = wl.step_q(step, 0)
        gpu.append(0, ks, vs)
        orc.append(0, to_f64(ks[pick]), to_f64(vs[pick]))
        out = gpu.attend_and_score(0, q)
        ref = orc.attend_and_score(0, to_f64(q[pick]))
        assert_out_close(to_f64(out[pick]), ref, cfg.kv_dtype, f"step {step}")
        calls += 1
    T = 3
    ks, vs = zip(*[wl.step_kv(2 + j, 0) for j in range(T)])
    kc, vc = torch.cat(ks, dim=1), torch.cat(vs, dim=1)
    gpu.append(0, kc, vc)
    orc.append(0, to_f64(kc[pick]), to_f64(vc[pick]))
    q = torch.stack([wl.step_q(2 + j, 0) for j in range(T)], dim=1).contiguous()
    out = gpu.attend_and_score_chunk(0, q)
    ref = orc.attend_and_score_chunk(0, to_f64(q[pick]))
    for j in range(T):
        assert_out_close(to_f64(out[pick, j]), ref[:, j], cfg.kv_dtype, f"chunk query {j}")
    calls += T
    nn = gpu.layer_length(0)
    ss = 1.0 / (cfg.n_layers * cfg.n_q_heads)
    assert_scores_close(gpu.get_scores()[pick], orc.score, nn, calls * cfg.n_q_heads * ss)
    gpu.close()


def test_prod_shape_subset_of_sequences():
    # 16384-token context, int4-g32 T2; 4 of the 64 sequences (sequences are independent units of work)
    _run_shape(dataclasses.replace(CONFIGS["prod"], n_layers=1, batch=4, decode_steps=2), "lazy", steps_after=1)


def test_decode_step_equals_per_layer_calls():
    """tkv_decode_step is tkv_append + tkv_attend_and_score per layer: same bits."""
    from gpu_common import Pair
    cfg = small_config(n_layers=3, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, kv_dtype="bf16", context=500,
                       decode_steps=4)
    a, b = Pair(cfg), Pair(cfg)
    k_all, v_all, q_all = a.wl.decode_inputs(0, 4)
    for s in range(4):
        oa = a.gpu.decode_step(k_all[s], v_all[s], q_all[s])
        for l in range(cfg.n_layers):
            b.gpu.append(l, k_all[s, l], v_all[s, l])
            ob = b.gpu.attend_and_score(l, q_all[s, l])
            assert torch.equal(oa[l], ob)
        if s == 1:
            for p in (a, b):
                p.gpu.classify(cfg.policy_ppm)
                p.gpu.migrate()
    assert np.array_equal(a.gpu.get_scores().view(np.uint32), b.gpu.get_scores().view(np.uint32))
    assert np.array_equal(a.gpu.get_tiers(), b.gpu.get_tiers())
    a.close(); b.close()


# Whole steps of which some pairs go in parts (how many parts, pairs in parts, mode, scorer, shape) and steps and single calls of
# whole pairs with logits beyond the LDS: test_abi_host.py holds the launches to it.
STEPS_IN_PARTS = [
    (3, 24, "lazy", "attention", dict(n_layers=4, batch=70, n_q_heads=5, n_kv_heads=1, head_dim=128, context=700)),          # list lengths from device counters
    (3, 32, "wait", "vatp", dict(n_layers=9, batch=4, n_q_heads=8, n_kv_heads=8, head_dim=64, context=1300)),
    (2, 100, "lazy", "combined", dict(n_layers=25, batch=1, n_q_heads=24, n_kv_heads=4, head_dim=128, context=800, t2_format="int4_g32", kv_dtype="f16")),   # all pairs
    (3, 80, "lazy", "attention", dict(n_layers=28, batch=3, n_q_heads=28, n_kv_heads=4, head_dim=128, context=2900)),        # score tiles of 64 columns
    (2, 102, "wait", "redundancy", dict(n_layers=34, batch=1, n_q_heads=6, n_kv_heads=3, head_dim=64, context=1700)),        # three kv heads
    (4, 32, "lazy", "vatp", dict(n_layers=9, batch=4, n_q_heads=8, n_kv_heads=8, head_dim=64, context=2040, t2_format="int4_g32")),
    (5, 48, "lazy", "attention", dict(n_layers=28, batch=5, n_q_heads=28, n_kv_heads=4, head_dim=128, context=2490)),
    (6, 24, "wait", "combined", dict(n_layers=20, batch=7, n_q_heads=8, n_kv_heads=2, head_dim=64, context=3060, kv_dtype="f16")),
    (7, 24, "lazy", "attention", dict(n_layers=4, batch=70, n_q_heads=5, n_kv_heads=1, head_dim=128, context=1780, t2_format="int4_g32", kv_dtype="f16")),
    (8, 24, "lazy", "redundancy", dict(n_layers=4, batch=70, n_q_heads=5, n_kv_heads=1, head_dim=128, context=2040)),
    (8, 24, "lazy", "vatp", dict(n_layers=4, batch=70, n_q_heads=5, n_kv_heads=1, head_dim=128, context=90, decode_steps=1950)),   # fewer tiles than parts
    (4, 32, "lazy", "attention", dict(n_layers=9, batch=4, n_q_heads=8, n_kv_heads=8, head_dim=64, context=40, decode_steps=2000)),   # ... of list lengths from the arguments
]
STEPS_BEYOND_THE_LDS = [
    dict(n_layers=7, batch=24, n_q_heads=64, n_kv_heads=8, head_dim=64, context=2900),
    dict(n_layers=64, batch=1, n_q_heads=28, n_kv_heads=4, head_dim=128, context=3500, t2_format="int4_g32"),
    dict(n_layers=32, batch=1, n_q_heads=48, n_kv_heads=8, head_dim=128, context=4000),
    dict(n_layers=11, batch=3, n_q_heads=64, n_kv_heads=8, head_dim=64, context=2900),
]
CALLS_BEYOND_THE_LDS = [
    dict(batch=32, n_q_heads=64, n_kv_heads=8, head_dim=64, context=2900, sequences=2),
    dict(batch=64, n_q_heads=28, n_kv_heads=4, head_dim=128, context=3500, t2_format="int4_g32", sequences=2),
]
PRECISION = dict(n_layers=32, batch=1, n_q_heads=40, n_kv_heads=8, head_dim=128, context=6001, decode_steps=2)


@pytest.mark.parametrize("mode,scorer,shape", [
    # split pairs (fewer than 96 pairs in the step)
    ("wait", "combined", dict(n_layers=5, batch=3, n_q_heads=10, n_kv_heads=2, head_dim=128, context=700)),
    ("lazy", "attention", dict(n_layers=40, batch=1, n_q_heads=5, n_kv_heads=1, head_dim=128, context=333)),    # two passes of the finishing kernel
    ("lazy", "vatp", dict(n_layers=2, batch=8, n_q_heads=24, n_kv_heads=4, head_dim=64, context=129, kv_dtype="f32")),
    # one workgroup per pair
    ("lazy", "attention", STEPS_BEYOND_THE_LDS[0]),
    ("wait", "vatp", dict(n_layers=40, batch=1, n_q_heads=28, n_kv_heads=4, head_dim=128, context=333, t2_format="int4_g32")),
    ("wait", "attention", dict(n_layers=4, batch=70, n_q_heads=4, n_kv_heads=2, head_dim=64, context=200)),
    ("lazy", "redundancy", dict(n_layers=3, batch=9, n_q_heads=40, n_kv_heads=8, head_dim=128, context=31, kv_dtype="f16")),
    ("lazy", "attention", dict(n_layers=70, batch=1, n_q_heads=6, n_kv_heads=2, head_dim=64, context=65, t2_format="int4_g32")),   # two groups of layers
    ("lazy", "vatp", STEPS_BEYOND_THE_LDS[1]),                                                                       # ... value norms
    ("wait", "redundancy", STEPS_BEYOND_THE_LDS[2]),                                                                 # ... the penalty
    ("lazy", "combined", dict(n_layers=12, batch=1, n_q_heads=8, n_kv_heads=8, head_dim=128, context=300)),
    ("lazy", "attention", dict(n_layers=6, batch=2, n_q_heads=32, n_kv_heads=8, head_dim=128, context=300, t2_format="int4_g32", kv_dtype="f16")),
])
def test_decode_step_serves_several_layers_per_launch(mode, scorer, shape):
    """A decode step's launches serve groups of layers, against per-layer calls: also right behind a re-tiering whose
    transfers are in flight (lazy: some layers read their rows' old slots; wait: layers that wait for their prefetch go in
    small groups), where a step takes several groups, and above 64 sequences.  Where pairs are split as in single calls
    the bits are the same.  With one workgroup per pair the same products are added in another order: outputs within 1e-5
    of the head's largest value and scores within 1e-5 of the magnitudes added, the bounds a single call keeps against
    the oracle for binary32 rows (each side's rounding is a few 1e-7)."""
    import paper_2605_09490_amd as tkv
    from tkv_synth import Workload
    cfg = small_config(name="groups", **{**dict(kv_dtype="bf16", decode_steps=4, k_window=16, policy_ppm=(300_000, 400_000, 250_000, 50_000)), **shape})
    same_bits = cfg.kv_dtype == "f32" or cfg.n_layers * cfg.batch * cfg.n_kv_heads < 96
    print(f"[case] {mode} {scorer} {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    kv = [tkv.TieredKV(cfg.n_layers, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens, kv_dtype=cfg.kv_dtype,
                       t2_format=cfg.t2_format, k_window=16, prefetch_mode=mode, scorer=scorer) for _ in range(2)]
    for l in range(cfg.n_layers):
        k, v = wl.context_kv(l)
        for c in kv:
            c.append(l, k, v)
    k_all, v_all, q_all = wl.decode_inputs(0, 4)
    for s in range(4):
        oa = kv[0].decode_step(k_all[s], v_all[s], q_all[s])
        for l in range(cfg.n_layers):
            kv[1].append(l, k_all[s, l], v_all[s, l])
            ob = kv[1].attend_and_score(l, q_all[s, l])
            if same_bits:
                assert torch.equal(oa[l], ob), (s, l)
            else:
                assert ((oa[l] - ob).abs() <= 1e-5 * ob.abs().amax(-1, keepdim=True)).all(), (s, l)
        sa, sb = (c.get_scores() for c in kv)
        if same_bits:
            assert np.array_equal(sa.view(np.uint32), sb.view(np.uint32)), s
        else:
            # a penalised score is a difference of magnitudes of at most about 1 / cache length per step each
            floor = 1e-5 * (s + 1) / cfg.context if scorer == "redundancy" else 1e-9
            assert (np.abs(sa - sb) <= 1e-5 * np.abs(sb) + floor).all(), s
        if s in (0, 2):
            kv[0].classify(cfg.policy_ppm)
            kv[1].set_tiers(kv[0].get_pending_tiers())     # scores that differ in the last bit may rank differently
            for c in kv:
                c.migrate()
    for c in kv:
        c.close()


@pytest.mark.parametrize("mode,scorer,shape", [t[2:] for t in STEPS_IN_PARTS])
def test_decode_step_whose_last_pairs_go_in_parts(mode, scorer, shape):
    """The pairs of a round that the chip does not fill are walked in parts and their weights and outputs made by the score
    launch: the same comparison with per-layer calls, with the same bounds, at numbers of pairs and tokens where that is done."""
    test_decode_step_serves_several_layers_per_launch(mode, scorer, shape)


@pytest.mark.parametrize("shape", [
    dict(n_layers=28, batch=1, n_q_heads=28, n_kv_heads=4, head_dim=128, context=3100),                    # pairs in two parts
    dict(n_layers=3, batch=70, n_q_heads=4, n_kv_heads=2, head_dim=64, context=150, kv_dtype="f16"),       # list lengths from device counters
    dict(n_layers=4, batch=64, n_q_heads=24, n_kv_heads=4, head_dim=128, context=90, t2_format="int4_g32"),   # WAIT: layers one by one
    dict(n_layers=5, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, context=700),                      # split pairs
    dict(n_layers=4, batch=70, n_q_heads=5, n_kv_heads=1, head_dim=128, context=2040),                     # 24 of the last layer's 70 pairs in eight parts
    STEPS_BEYOND_THE_LDS[3],                                                                               # 8 of its 24 in six
    dict(n_layers=3, batch=130, n_q_heads=4, n_kv_heads=2, head_dim=64, context=300),                      # vector instructions
])
def test_prop1_of_whole_steps(shape, monkeypatch):
    """T1 placement, prefetch mode and the memory there is for a step's scratch change no bit of a decode step: the same rows
    in T1 with attention reading old slots while the copies are in flight (LAZY), behind them (WAIT: small groups of
    layers), with the rows in T0 all along, and with every allocation refused that the cache can do without (one layer per
    launch, parts of pairs among them).  Steps straddle two plans."""
    import paper_2605_09490_amd as tkv
    from tkv_synth import Workload
    cfg = small_config(name="prop1", **{**dict(kv_dtype="bf16", decode_steps=6, k_window=16, sigma=1.0), **shape})
    print(f"[case] {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    empty, pinned = torch.empty, []

    def scarce(*a, **kw):                 # the pinned store is the last thing a cache must have
        if kw.get("pin_memory"):
            pinned.append(1)
        elif pinned:
            raise RuntimeError("refused")
        return empty(*a, **kw)

    def cache(mode, refuse=False):
        with monkeypatch.context() as m:
            if refuse:
                m.setattr(torch, "empty", scarce)
            return tkv.TieredKV(cfg.n_layers, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens,
                                kv_dtype=cfg.kv_dtype, t2_format=cfg.t2_format, k_window=16, prefetch_mode=mode)

    kv = {"lazy": cache("lazy"), "wait": cache("wait"), "all in T0": cache("lazy"), "scarce": cache("lazy", refuse=True)}
    assert kv["scarce"].get_stats()["device_bytes"] < kv["lazy"].get_stats()["device_bytes"]
    for l in range(cfg.n_layers):
        k, v = wl.context_kv(l)
        for c in kv.values():
            c.append(l, k, v)
    k_all, v_all, q_all = wl.decode_inputs(0, 6)
    rng = np.random.default_rng(11)
    tiers = rng.choice(4, size=(cfg.batch, cfg.context), p=(0.3, 0.4, 0.25, 0.05)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    for s in range(6):
        outs = {n: c.decode_step(k_all[s], v_all[s], q_all[s]) for n, c in kv.items()}
        scores = {n: c.get_scores().view(np.uint32) for n, c in kv.items()} if s != 2 else None   # (reading them waits)
        for n in kv:
            assert torch.equal(outs[n], outs["lazy"]), (s, n)
            assert scores is None or np.array_equal(scores[n], scores["lazy"]), (s, n)
        if s in (1, 3):
            for n, c in kv.items():
                c.set_tiers(np.where(tiers == 1, 0, tiers) if n == "all in T0" else tiers)
                c.migrate()
            swap = (tiers <= 1) & (rng.random(tiers.shape) < 0.3)
            swap[:, :4] = False
            swap[:, -16:] = False
            tiers = np.where(swap, 1 - tiers, tiers).astype(np.uint8)
    assert kv["wait"].get_stats()["attend_waits"] > 0
    assert kv["lazy"].get_stats()["lazy_old_reads"] > 0
    for c in kv.values():
        c.close()


@pytest.mark.parametrize("shape", [
    dict(batch=64, n_q_heads=28, n_kv_heads=4, head_dim=128, context=97),
    dict(batch=130, n_q_heads=4, n_kv_heads=2, head_dim=64, context=129, t2_format="int4_g32", kv_dtype="f16"),   # list lengths from device counters; few heads
    dict(batch=256, n_q_heads=1, n_kv_heads=1, head_dim=64, context=65),                                           # ... one, two tiles
    dict(batch=86, n_q_heads=6, n_kv_heads=3, head_dim=64, context=1021, sequences=2),                             # ... two, the longest lists on the vector ALUs
    dict(batch=86, n_q_heads=6, n_kv_heads=3, head_dim=64, context=1022, t2_format="int4_g32", sequences=2),       # ... the shortest on the matrix cores
    *CALLS_BEYOND_THE_LDS,                                                                                         # the second: the production batch's kernel
])
def test_single_calls_with_a_pair_for_every_compute_unit(shape):
    """256 or more pairs: single calls take one workgroup per pair as a whole step does.  Outputs and scores against the
    oracle, and the same bits from tkv_decode_step and from the call that allocates nothing (where its array is large
    enough), before and after a re-tiering."""
    from gpu_common import Pair, assert_out_close, assert_scores_close, to_f64
    import paper_2605_09490_amd as tkv
    shape = dict(shape)
    check = shape.pop("sequences", None)      # sequences compared with the oracle (they are independent); None: all
    cfg = small_config(name="pairs", n_layers=1, decode_steps=3, k_window=16, policy_ppm=(300_000, 400_000, 250_000, 50_000),
                       **{**dict(kv_dtype="bf16"), **shape})
    print(f"[case] {shape}", flush=True)
    p = Pair(cfg, prefetch_mode="lazy") if check is None else None
    if p is None:
        p = Pair(dataclasses.replace(cfg, batch=check), prefetch_mode="lazy", preload=False)
        p.gpu.close()
        from tkv_synth import Workload
        p.wl = Workload(cfg, device="cuda")
    def cache():
        return tkv.TieredKV(1, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens, kv_dtype=cfg.kv_dtype,
                            t2_format=cfg.t2_format, k_sink=cfg.k_sink, k_window=cfg.k_window, score_scale=p.score_scale,
                            prefetch_mode="lazy")
    nb = check or cfg.batch
    ctx = p.wl.context_kv(0)
    gpus = [cache() for _ in range(3)]
    for g in gpus:
        g.append(0, *ctx)
    if check is not None:
        p.orc.append(0, to_f64(ctx[0][:nb]), to_f64(ctx[1][:nb]))
    for step in range(3):
        k, v = p.wl.step_kv(step, 0)
        q = p.wl.step_q(step, 0)
        p.orc.append(0, to_f64(k[:nb]), to_f64(v[:nb]))
        ref = p.orc.attend_and_score(0, to_f64(q[:nb]))
        gpus[0].append(0, k, v)
        out = gpus[0].attend_and_score(0, q)
        assert_out_close(to_f64(out[:nb]), ref, cfg.kv_dtype, f"step {step}")
        assert torch.equal(out, gpus[1].decode_step(k[None], v[None], q[None])[0])
        gpus[2].append(0, k, v)
        try:
            assert torch.equal(out, gpus[2].attend_and_score_noalloc(0, q, torch.full_like(out, float("nan"))))
        except tkv.TkvError as e:
            assert e.status == tkv.TKV_ECAPACITY and cfg.batch * cfg.n_q_heads * cfg.max_tokens * 4 > 8 << 20
            gpus[2].attend_and_score(0, q)
        scores = [g.get_scores() for g in gpus]
        assert np.array_equal(scores[0].view(np.uint32), scores[1].view(np.uint32))
        assert np.array_equal(scores[0].view(np.uint32), scores[2].view(np.uint32))
        if step == 0:
            n = gpus[0].layer_length(0)
            gpus[0].classify(cfg.policy_ppm)
            plan = gpus[0].get_pending_tiers()[:, :n]
            for g in gpus[1:]:
                g.set_tiers(plan)
            for g in gpus:
                g.migrate()
            p.orc.set_tiers(plan[:nb])
            p.orc.migrate()
    assert_scores_close(gpus[0].get_scores()[:nb], p.orc.score, gpus[0].layer_length(0), 3 * cfg.n_q_heads * p.score_scale)
    for g in gpus:
        g.close()
    p.close()


@pytest.mark.parametrize("n_q,shape", [
    (2, dict(batch=1, n_q_heads=16, n_kv_heads=2, head_dim=64, context=9001)),     # 16 splits per pair: one round of loads
    (2, dict(batch=1, n_q_heads=16, n_kv_heads=2, head_dim=64, context=9601)),     # more: a chain
    (4, dict(batch=1, n_q_heads=14, n_kv_heads=2, head_dim=128, context=4500)),    # 16 splits, two blocks of columns, four queries side by side
    (4, dict(batch=1, n_q_heads=14, n_kv_heads=2, head_dim=128, context=5200)),    # ... more
    (2, dict(batch=1, n_q_heads=14, n_kv_heads=2, head_dim=128, context=9800)),    # more than 16 splits of 16 tiles, one block of columns
    (3, dict(batch=32, n_q_heads=16, n_kv_heads=2, head_dim=64, context=600)),     # no room for four side by side: two
    (4, dict(batch=32, n_q_heads=28, n_kv_heads=4, head_dim=128, context=300)),    # ... one
    (13, dict(batch=32, n_q_heads=3, n_kv_heads=3, head_dim=64, context=300)),     # many queries in one launch
    (16, dict(batch=1, n_q_heads=128, n_kv_heads=128, head_dim=128, context=150)), # ... of more heads than the score launch has LDS for
])
def test_chunks_by_split_count_and_queries_side_by_side(n_q, shape):
    """The finishing kernel of a chunk in each of its launch shapes: outputs and scores of a chunk over all four tiers
    against the oracle."""
    from gpu_common import Pair, assert_out_close, assert_scores_close
    cfg = small_config(name="chunk", n_layers=1, kv_dtype="bf16", decode_steps=n_q, k_window=16, sigma=1.0, **shape)
    print(f"[case] chunk of {n_q}, {shape}", flush=True)
    p = Pair(cfg, prefetch_mode="lazy")
    tiers = np.random.default_rng(3).choice(4, size=(cfg.batch, cfg.context), p=(0.4, 0.3, 0.2, 0.1)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    p.force_tiers(tiers)
    ks, vs = zip(*[p.wl.step_kv(j, 0) for j in range(n_q)])
    p.append(0, torch.cat(ks, dim=1), torch.cat(vs, dim=1))
    got, ref = p.attend_chunk(0, torch.stack([p.wl.step_q(j, 0) for j in range(n_q)], dim=1).contiguous())
    for j in range(n_q):
        assert_out_close(got[:, j], ref[:, j], cfg.kv_dtype, f"query {j}")
    n = cfg.context + n_q
    assert_scores_close(p.gpu.get_scores(), p.orc.score, n, n_q * cfg.n_q_heads * p.score_scale)
    p.close()


@pytest.mark.parametrize("n_q,kv_dtype,t2,scorer,shape", [
    (17, "bf16", "int8_row", "attention", dict(batch=2, n_q_heads=2, n_kv_heads=2, head_dim=128, context=31)),     # G = 1, one group; a list of one tile
    (33, "f16", "int4_g32", "attention", dict(batch=2, n_q_heads=3, n_kv_heads=1, head_dim=64, context=333)),      # 32 tokens in a launch, one behind them
    (7, "bf16", "int4_g32", "combined", dict(batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, context=1500)),    # 35 columns: the second group nearly empty
    (13, "f16", "int8_row", "vatp", dict(batch=3, n_q_heads=45, n_kv_heads=9, head_dim=128, context=700)),         # nine kv heads, 65 columns: more blocks than a wave keeps
    (20, "bf16", "int8_row", "attention", dict(batch=1, n_q_heads=7, n_kv_heads=1, head_dim=128, context=6100)),   # more than 16 splits per pair
    (5, "bf16", "int4_g32", "attention", dict(batch=1, n_q_heads=16, n_kv_heads=2, head_dim=64, context=2500)),    # five to 16 splits, 64-row tiles
    (6, "bf16", "int8_row", "attention", dict(batch=66, n_q_heads=7, n_kv_heads=1, head_dim=64, context=190)),     # list lengths from the device counters
    (32, "bf16", "int8_row", "attention", dict(batch=4, n_q_heads=128, n_kv_heads=128, head_dim=64, context=2300)),   # 68 KB of dynamic LDS, two runs of tiles
])
def test_chunks_whose_logits_are_not_written(n_q, kv_dtype, t2, scorer, shape):
    """More columns (query token, head) than one group of a workgroup takes: outputs and scores of a chunk over all four
    tiers against the oracle, at the edges of column groups, list runs and split counts.  Tolerances as everywhere: the
    products are exact in 16 bits and added in binary32."""
    from gpu_common import Pair, assert_out_close, assert_scores_close
    cfg = small_config(name="chunk", n_layers=1, kv_dtype=kv_dtype, t2_format=t2, decode_steps=n_q, k_window=8, sigma=1.0, **shape)
    print(f"[case] chunk of {n_q}, {kv_dtype} {t2} {scorer}, {shape}", flush=True)
    p = Pair(cfg, prefetch_mode="lazy", scorer=scorer)
    tiers = np.random.default_rng(5).choice(4, size=(cfg.batch, cfg.context), p=(0.4, 0.3, 0.2, 0.1)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -8:] = 0
    p.force_tiers(tiers)
    ks, vs = zip(*[p.wl.step_kv(j, 0) for j in range(n_q)])
    p.append(0, torch.cat(ks, dim=1), torch.cat(vs, dim=1))
    got, ref = p.attend_chunk(0, torch.stack([p.wl.step_q(j, 0) for j in range(n_q)], dim=1).contiguous())
    for j in range(n_q):
        assert_out_close(got[:, j], ref[:, j], kv_dtype, f"query {j}")
    total = n_q * cfg.n_q_heads * p.score_scale if scorer == "attention" else float(p.orc.score_mag.sum(axis=1).max())
    assert_scores_close(p.gpu.get_scores(), p.orc.score, cfg.context + n_q, total, mag64=p.orc.score_mag)
    p.close()


def _chunk_pair(cfg, tiers, k, v, k_new, v_new):
    """A one-layer cache and its oracle over the given context rows, tiers forced, with the chunk's rows appended."""
    from gpu_common import Pair
    p = Pair(cfg, prefetch_mode="lazy", preload=False)
    p.append(0, k, v)
    p.force_tiers(tiers)
    p.append(0, k_new, v_new)
    return p


def _step_rows(wl, n_q):
    ks, vs = zip(*[wl.step_kv(j, 0) for j in range(n_q)])
    return torch.cat(ks, dim=1), torch.cat(vs, dim=1), torch.stack([wl.step_q(j, 0) for j in range(n_q)], dim=1).contiguous()


@pytest.mark.parametrize("n_q,heads,dim,kv_dtype,t2", [
    (13, 7, 128, "bf16", "int8_row"),      # 91 columns: five past the last in the last block
    (9, 5, 64, "f16", "int4_g32"),         # 45 columns
    (3, 5, 128, "f16", "int8_row"),        # 15 columns: logits written
])
def test_chunk_over_keys_with_infinities(n_q, heads, dim, kv_dtype, t2):
    """A key row with an element of -inf that every query multiplies by a positive number has a logit of -inf and no weight.
    Its score stays what it was: the columns past a chunk's last (zeros times infinity) have no part in it."""
    from gpu_common import assert_out_close, assert_scores_close
    from tkv_synth import Workload
    cfg = small_config(name="inf", n_layers=1, batch=2, n_q_heads=heads, n_kv_heads=1, head_dim=dim, kv_dtype=kv_dtype,
                       t2_format=t2, context=700, decode_steps=n_q, k_window=16, sigma=1.0)
    print(f"[case] infinite keys, chunk of {n_q}, {heads} heads, {dim}, {kv_dtype}", flush=True)
    wl = Workload(cfg, device="cuda")
    k, v = wl.context_kv(0)
    k_new, v_new, q = _step_rows(wl, n_q)
    q[..., 3] = q[..., 3].abs() + 0.5
    rows = [5, 100, 350, 690]
    k[:, rows, :, 3] = float("-inf")
    tiers = np.random.default_rng(7).choice(4, size=(cfg.batch, cfg.context), p=(0.4, 0.3, 0.2, 0.1)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    tiers[:, rows] = (0, 0, 1, 0)
    p = _chunk_pair(cfg, tiers, k, v, k_new, v_new)
    got, ref = p.attend_chunk(0, q)
    assert_out_close(got, ref, kv_dtype)
    scores = p.gpu.get_scores()
    assert (scores[:, rows] == 0).all(), scores[:, rows]
    assert_scores_close(scores, p.orc.score, cfg.context + n_q, n_q * heads * p.score_scale)
    p.close()


@pytest.mark.parametrize("every", [1, 9])
@pytest.mark.parametrize("n_q,heads,dim,t2", [
    (3, 5, 128, "int8_row"),               # 15 columns, one block, logits written
    (5, 5, 64, "int4_g32"),                # 25 columns, two blocks
    (9, 5, 128, "int4_g32"),               # 45 columns: logits not written
    (13, 7, 64, "int8_row"),
])
def test_chunk_over_large_values_in_binary16(n_q, heads, dim, t2, every):
    """T2 rows of a binary16 cache whose V scales are far above one (int8 rows up to some 5000, int4 groups up to 200 and 8000):
    the weight times such a scale does not fit binary16 beside the weights' own shift.  Every row, or every ninth."""
    from gpu_common import assert_out_close, assert_scores_close
    from tkv_synth import Workload
    cfg = small_config(name="large", n_layers=1, batch=2, n_q_heads=heads, n_kv_heads=1, head_dim=dim, kv_dtype="f16",
                       t2_format=t2, context=900, decode_steps=n_q, k_window=16, sigma=1.0)
    wl = Workload(cfg, device="cuda")
    k, v = wl.context_kv(0)
    k_new, v_new, q = _step_rows(wl, n_q)
    tiers = np.random.default_rng(11).choice(4, size=(cfg.batch, cfg.context), p=(0.2, 0.1, 0.6, 0.1)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    for amp in (2.0, 100.0, 2000.0):
        print(f"[case] values of {amp}, chunk of {n_q}, {heads} heads, {dim}, {t2}, every {every}", flush=True)
        vv = v.clone()
        vv[:, ::every] *= amp
        p = _chunk_pair(cfg, tiers, k, vv, k_new, v_new)
        got, ref = p.attend_chunk(0, q)
        print(f"[case] worst error {assert_out_close(got, ref, 'f16', f'values of {amp}'):.2e} of the head max-norm", flush=True)
        assert_scores_close(p.gpu.get_scores(), p.orc.score, cfg.context + n_q, n_q * heads * p.score_scale)
        p.close()


@pytest.mark.parametrize("heads,dim,kv_dtype,t2,context,batch", [
    (7, 128, "bf16", "int4_g32", 300, 256),        # one workgroup per pair
    (5, 128, "f16", "int8_row", 290, 256),
    (8, 64, "f16", "int4_g32", 321, 256),
    (1, 64, "bf16", "int8_row", 257, 256),
    (7, 128, "bf16", "int8_row", 1500, 2),         # pairs split, matrix instructions
    (4, 128, "f16", "int4_g32", 261, 3),
    (8, 128, "f16", "int8_row", 1025, 2),
    (3, 128, "bf16", "int4_g32", 700, 2),          # ... vector instructions
])
def test_single_calls_over_infinite_keys_and_large_values(heads, dim, kv_dtype, t2, context, batch):
    """Rows whose logit is -inf have no weight and keep their score, padding columns have no part in anything, T2 rows with V
    scales far above one stay in binary16's range, and queries may begin at any element."""
    from gpu_common import assert_out_close, assert_scores_close
    from tkv_synth import Workload
    cfg = small_config(name="pairs-edge", n_layers=1, batch=batch, n_q_heads=heads, n_kv_heads=1, head_dim=dim, kv_dtype=kv_dtype,
                       t2_format=t2, context=context, decode_steps=1, k_window=16, sigma=1.0)
    wl = Workload(cfg, device="cuda")
    k, v = wl.context_kv(0)
    k_new, v_new, _ = _step_rows(wl, 1)
    q = wl.step_q(0, 0)
    q[..., 3] = q[..., 3].abs() + 0.5
    rows = [5, 100, 250]
    k[:, rows, :, 3] = float("-inf")
    tiers = np.random.default_rng(7).choice(4, size=(cfg.batch, context), p=(0.3, 0.2, 0.4, 0.1)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    tiers[:, rows] = (0, 1, 0)
    offset = torch.empty(q.numel() + 1, dtype=q.dtype, device="cuda")[1:].view(q.shape).copy_(q)
    for amp in (1.0, 2000.0):
        print(f"[case] {batch} pairs, {heads} heads, {dim}, {kv_dtype}, {t2}, values of {amp}", flush=True)
        vv = v.clone()
        vv[:, ::9] *= amp
        p = _chunk_pair(cfg, tiers, k, vv, k_new, v_new)
        got, ref = p.attend(0, offset)
        assert_out_close(got, ref, kv_dtype, f"values of {amp}")
        scores = p.gpu.get_scores()
        assert (scores[:, rows] == 0).all(), scores[:, rows]
        assert_scores_close(scores, p.orc.score, context + 1, heads * p.score_scale)
        p.close()


def _one_token_outputs(kind, cfg, k, v, k_new, v_new, q, tiers=None):
    """Outputs [layers, sequences, heads, head_dim] and scores of one decode step by whole steps ("step"), per-layer calls
    ("call") or chunks of two query tokens ("chunk": the last one's) over the context rows k[l], v[l] and the new row."""
    import paper_2605_09490_amd as tkv
    kv = tkv.TieredKV(cfg.n_layers, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens, kv_dtype=cfg.kv_dtype,
                      t2_format=cfg.t2_format, k_window=16, prefetch_mode="lazy")
    last = 1 if kind == "chunk" else 0        # a chunk's first query token stands before the new row
    for l in range(cfg.n_layers):
        kv.append(l, k[l], v[l])
    if tiers is not None:
        kv.set_tiers(tiers)
        kv.migrate()
    if kind == "step":
        out = kv.decode_step(k_new, v_new, q)
    else:
        outs = []
        for l in range(cfg.n_layers):
            kn, vn = k_new[l], v_new[l]
            if last:
                kn, vn = torch.cat([kn, kn], dim=1), torch.cat([vn, vn], dim=1)
            kv.append(l, kn, vn)
            if last:
                outs.append(kv.attend_and_score_chunk(l, torch.stack([q[l], q[l]], dim=1).contiguous())[:, 1])
            else:
                outs.append(kv.attend_and_score(l, q[l]))
        out = torch.stack(outs)
    scores = kv.get_scores()
    kv.close()
    return out, scores


ONE_TOKEN_LAUNCHES = [
    ("call", dict(n_layers=1, batch=256, n_q_heads=7, n_kv_heads=1, head_dim=128, context=300)),                      # one workgroup per pair
    ("call", dict(n_layers=1, batch=128, n_q_heads=16, n_kv_heads=2, head_dim=64, context=321, kv_dtype="f16")),
    ("call", dict(n_layers=1, batch=128, n_q_heads=4, n_kv_heads=2, head_dim=64, context=333)),                       # ... vector instructions
    ("step", dict(n_layers=64, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, context=200, kv_dtype="f16")),      # ... of whole steps
    ("step", dict(n_layers=25, batch=2, n_q_heads=14, n_kv_heads=2, head_dim=128, context=1500)),                     # pairs in parts
    ("call", dict(n_layers=2, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, context=700)),                       # pairs split, matrix instructions
    ("call", dict(n_layers=2, batch=2, n_q_heads=8, n_kv_heads=2, head_dim=128, context=1100, kv_dtype="f16")),
    ("call", dict(n_layers=2, batch=2, n_q_heads=6, n_kv_heads=2, head_dim=128, context=700)),                        # ... vector instructions
    ("call", dict(n_layers=2, batch=2, n_q_heads=16, n_kv_heads=2, head_dim=64, context=900, kv_dtype="f16")),
]


@pytest.mark.parametrize("kind,shape", ONE_TOKEN_LAUNCHES + [("chunk", ONE_TOKEN_LAUNCHES[5][1])])
def test_logits_that_are_no_numbers_reach_the_output(kind, shape):
    """A NaN in a key row, and an infinite key element under a query element of zero: the heads that read the row have no
    number for an output, whichever launch serves the call.  All others have the bits they have without."""
    from tkv_synth import Workload
    cfg = small_config(name="nan", **{**dict(kv_dtype="bf16", decode_steps=2, k_window=16, sigma=1.0), **shape})
    print(f"[case] {kind} {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    k, v = (list(x) for x in zip(*(wl.context_kv(l) for l in range(cfg.n_layers))))
    k_all, v_all, q_all = wl.decode_inputs(0, 1)
    q, G = q_all[0].clone(), cfg.n_q_heads // cfg.n_kv_heads
    q[-1, -1, -G:, 5] = 0
    clean, _ = _one_token_outputs(kind, cfg, k, v, k_all[0], v_all[0], q)
    k[0], k[-1] = k[0].clone(), k[-1].clone()
    k[0][0, 17, 0, 3] = float("nan")                    # first layer, sequence and kv head
    k[-1][-1, 130, -1, 5] = float("inf")                # last ones
    out, scores = _one_token_outputs(kind, cfg, k, v, k_all[0], v_all[0], q)
    hit = torch.zeros(clean.shape[:3], dtype=torch.bool, device="cuda")
    hit[0, 0, :G] = True
    hit[-1, -1, -G:] = True
    assert torch.isfinite(clean).all()
    assert out[hit].isnan().all(), int(out[hit].isfinite().sum())
    assert torch.equal(out[~hit], clean[~hit])
    assert np.isnan(scores[0, 17]) and np.isnan(scores[-1, 130])


@pytest.mark.parametrize("kind,shape", ONE_TOKEN_LAUNCHES + [
    ("call", dict(n_layers=2, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=64, context=700, kv_dtype="f32")),
    ("call", dict(n_layers=2, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, context=900, kv_dtype="f32")),
    ("chunk", ONE_TOKEN_LAUNCHES[5][1]),
])
def test_whole_tiles_of_keys_without_weight(kind, shape):
    """Rows whose logit is -inf, whole tiles of them, a list's first and others: no weight, whatever else a wave walks."""
    from gpu_common import assert_out_close, to_f64
    from tkv_synth import Workload
    cfg = small_config(name="tiles", **{**dict(kv_dtype="bf16", decode_steps=2, k_window=16, sigma=1.0), **shape})
    cfg = dataclasses.replace(cfg, recipe="bias")
    print(f"[case] {kind} {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    k, v = (list(x) for x in zip(*(wl.context_kv(l) for l in range(cfg.n_layers))))
    k_all, v_all, q_all = wl.decode_inputs(0, 1)
    q, G = q_all[0].clone(), cfg.n_q_heads // cfg.n_kv_heads
    q[..., 3] = q[..., 3].abs() + 0.5
    k[0] = k[0].clone()
    k[0][0, :192, :, 3] = float("-inf")
    out, scores = _one_token_outputs(kind, cfg, k, v, k_all[0], v_all[0], q)
    for kvh in range(cfg.n_kv_heads):
        kk, vv = (np.concatenate([to_f64(c[0][0, 192:, kvh]), to_f64(n[0, 0, 0, :, kvh])] + [to_f64(n[0, 0, 0, :, kvh])] * (kind == "chunk"))
                  for c, n in ((k, k_all), (v, v_all)))
        x = to_f64(q[0, 0, kvh * G:(kvh + 1) * G]) @ kk.T / np.sqrt(cfg.head_dim)
        w = np.exp(x - x.max(1, keepdims=True))
        assert_out_close(to_f64(out[0, 0, kvh * G:(kvh + 1) * G]), (w / w.sum(1, keepdims=True)) @ vv, cfg.kv_dtype)
    assert out.isfinite().all() and np.isfinite(scores).all()


@pytest.mark.parametrize("kind,shape", ONE_TOKEN_LAUNCHES)
def test_infinite_values_reach_the_output(kind, shape):
    """A value row with infinite elements at full precision: those elements of the outputs are infinite, whatever the row's
    weight (the largest one's, exactly 1 before it is normalised, or any other), the others what they are in 64 bits."""
    from gpu_common import assert_out_close, to_f64
    from tkv_synth import Workload
    cfg = small_config(name="infinite", **{**dict(kv_dtype="bf16", decode_steps=2, k_window=16, sigma=1.0), **shape})
    cfg = dataclasses.replace(cfg, recipe="bias")       # (no weight underflows)
    print(f"[case] {kind} {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    k, v = (list(x) for x in zip(*(wl.context_kv(l) for l in range(cfg.n_layers))))
    k_all, v_all, q_all = wl.decode_inputs(0, 1)
    q, G = q_all[0], cfg.n_q_heads // cfg.n_kv_heads
    for l, b, kvh in ((0, 0, 0), (cfg.n_layers - 1, cfg.batch - 1, cfg.n_kv_heads - 1)):
        v[l] = v[l].clone()
        x = to_f64(k[l][b, :, kvh]) @ to_f64(q[l, b, kvh * G:(kvh + 1) * G]).T
        for i, row in enumerate([*np.unique(x.argmax(0)), 7, 64, 101, cfg.context - 1]):
            v[l][b, row, kvh, 3 * i] = float("inf") if i % 2 else float("-inf")
    out, _ = _one_token_outputs(kind, cfg, k, v, k_all[0], v_all[0], q)
    for l, b, kvh in ((0, 0, 0), (cfg.n_layers - 1, cfg.batch - 1, cfg.n_kv_heads - 1)):
        kk, vv = (np.concatenate([to_f64(c[l][b, :, kvh]), to_f64(n[0, l, b, :, kvh])]) for c, n in ((k, k_all), (v, v_all)))
        x = to_f64(q[l, b, kvh * G:(kvh + 1) * G]) @ kk.T / np.sqrt(cfg.head_dim)
        w = np.exp(x - x.max(1, keepdims=True))
        w /= w.sum(1, keepdims=True)
        ref, inf = w @ np.where(np.isinf(vv), 0, vv), np.where(np.isinf(vv), vv, 0).sum(0)
        got = to_f64(out[l, b, kvh * G:(kvh + 1) * G])
        assert (got[:, inf != 0] == inf[inf != 0]).all(), got[:, inf != 0]
        assert_out_close(got[:, inf == 0], ref[:, inf == 0], cfg.kv_dtype)


@pytest.mark.parametrize("kind,t2,shape", [
    ("call", "int8_row", dict(n_layers=1, batch=256, n_q_heads=7, n_kv_heads=1, head_dim=128, context=300)),
    ("call", "int4_g32", dict(n_layers=1, batch=256, n_q_heads=5, n_kv_heads=1, head_dim=128, context=300, kv_dtype="f16")),
    ("call", "int4_g32", dict(n_layers=1, batch=256, n_q_heads=8, n_kv_heads=1, head_dim=64, context=300)),
    ("step", "int8_row", dict(n_layers=25, batch=2, n_q_heads=14, n_kv_heads=2, head_dim=128, context=1500, kv_dtype="f16")),
    ("call", "int8_row", dict(n_layers=2, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, context=700, kv_dtype="f16")),
    ("call", "int4_g32", dict(n_layers=2, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=128, context=700)),
    ("call", "int4_g32", dict(n_layers=2, batch=2, n_q_heads=6, n_kv_heads=2, head_dim=128, context=700)),       # vector instructions
])
def test_infinite_values_in_t2(kind, t2, shape):
    """A value row that is compressed with an element of -inf: its scale (int4: its group's) is infinite, the element's code the
    lowest, all others zero.  Code times scale is -inf there and no number in the rest of the row (group); elements of other
    groups have the bits that a finite row of the same codes gives them."""
    from tkv_synth import Workload
    cfg = small_config(name="infinite", **{**dict(kv_dtype="bf16", decode_steps=2, k_window=16, sigma=1.0, t2_format=t2), **shape})
    cfg = dataclasses.replace(cfg, recipe="bias")
    print(f"[case] {kind} {t2} {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    k, v = (list(x) for x in zip(*(wl.context_kv(l) for l in range(cfg.n_layers))))
    k_all, v_all, q_all = wl.decode_inputs(0, 1)
    G = cfg.n_q_heads // cfg.n_kv_heads
    v[0] = v[0].clone()
    v[0][0, 33, 0, 40] = float("-inf")
    tiers = np.random.default_rng(3).choice((0, 2), size=(cfg.batch, cfg.context)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    tiers[:, 33] = 2
    out, _ = _one_token_outputs(kind, cfg, k, v, k_all[0], v_all[0], q_all[0], tiers)
    got = out[0, 0, :G]
    lo, hi = (32, 64) if t2 == "int4_g32" else (0, cfg.head_dim)
    assert (got[:, 40] == float("-inf")).all(), got[:, 40]
    rest = torch.ones(cfg.head_dim, dtype=torch.bool, device="cuda")
    rest[lo:hi] = False
    assert got[:, rest].isfinite().all()
    rest = ~rest
    rest[40] = False
    assert got[:, rest].isnan().all()
    out[0, 0, :G] = 0
    assert out.isfinite().all()


@pytest.mark.parametrize("t2", ["int8_row", "int4_g32"])
@pytest.mark.parametrize("kind,shape", [
    ("call", dict(n_layers=1, batch=256, n_q_heads=5, n_kv_heads=1, head_dim=128, context=400)),
    ("call", dict(n_layers=1, batch=256, n_q_heads=8, n_kv_heads=1, head_dim=64, context=500)),
    ("call", dict(n_layers=2, batch=2, n_q_heads=14, n_kv_heads=2, head_dim=128, context=1500)),
    ("call", dict(n_layers=2, batch=2, n_q_heads=6, n_kv_heads=2, head_dim=128, context=1500)),      # vector instructions
])
def test_binary16_outputs_are_as_exact_whatever_the_values_magnitude(kind, t2, shape):
    """T2 rows of a binary16 cache whose values are far from one either way.  Outputs are linear in the values, so their error
    against 64 bits, relative to the outputs, is that of values of order one: a factor of two is left for another draw of the
    roundings (values of 1e-4 are rounded to fewer bits by binary16 itself, which the reference sees too)."""
    from gpu_common import to_f64
    from tkv_synth import Workload
    cfg = small_config(name="magnitude", **{**dict(kv_dtype="f16", decode_steps=2, k_window=16, t2_format=t2), **shape})
    cfg = dataclasses.replace(cfg, recipe="bias", sigma=1.5)
    print(f"[case] {kind} {t2} {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    tiers = np.random.default_rng(5).choice(4, size=(cfg.batch, cfg.context), p=(0.1, 0.05, 0.8, 0.05)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    k, v = (list(x) for x in zip(*(wl.context_kv(l) for l in range(cfg.n_layers))))
    k_new, v_new, _ = _step_rows(wl, 1)
    q = wl.step_q(0, 0)
    errs = []
    for amp in (1.0, 2.0 ** 11, 2.0 ** -13):
        p = _chunk_pair(dataclasses.replace(cfg, n_layers=1), tiers, k[0], v[0] * amp, k_new, v_new * amp)
        got, ref = p.attend(0, q)
        errs.append(float(np.linalg.norm(got - ref) / np.linalg.norm(ref)))
        print(f"[case] values of {amp}: error {errs[-1]:.2e}", flush=True)
        p.close()
    assert max(errs) <= 2 * errs[0], errs


@pytest.mark.parametrize("kind,shape", [
    ("call", dict(n_layers=1, batch=256, n_q_heads=5, n_kv_heads=1, head_dim=128, context=400)),
    ("call", dict(n_layers=1, batch=256, n_q_heads=8, n_kv_heads=1, head_dim=64, context=500)),
    ("call", dict(n_layers=2, batch=2, n_q_heads=14, n_kv_heads=2, head_dim=128, context=1500)),
    ("call", dict(n_layers=2, batch=2, n_q_heads=6, n_kv_heads=2, head_dim=128, context=1500)),      # vector instructions
])
def test_binary16_outputs_beside_a_row_with_nearly_all_the_attention(kind, shape):
    """A row that takes all of the attention but some 1e-3 to 1e-15 and has a value of zero, as first tokens often have: the
    outputs are made of weights far below the largest.  A logit's distance to that row's is rounded in binary32, and so is what
    it is the distance of: 2^-24 of it either time, beyond what the outputs are off without such a row."""
    from gpu_common import to_f64
    from tkv_synth import Workload
    cfg = small_config(name="sink", **{**dict(kv_dtype="f16", decode_steps=2, k_window=16), **shape})
    cfg = dataclasses.replace(cfg, recipe="bias", sigma=1.0)
    print(f"[case] {kind} {shape}", flush=True)
    wl = Workload(cfg, device="cuda")
    tiers = np.random.default_rng(5).choice(4, size=(cfg.batch, cfg.context), p=(0.4, 0.15, 0.4, 0.05)).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    k, v = wl.context_kv(0)
    k_new, v_new, _ = _step_rows(wl, 1)
    q = wl.step_q(0, 0)
    errs = []
    for logit in (0, 12, 24, 40):
        k[:, 2, :, 0], v[:, 2] = logit, 0
        p = _chunk_pair(dataclasses.replace(cfg, n_layers=1), tiers, k, v, k_new, v_new)
        got, ref = p.attend(0, q)
        errs.append(float(np.linalg.norm(got - ref) / np.linalg.norm(ref)))
        print(f"[case] logit {logit}: error {errs[-1]:.2e}", flush=True)
        p.close()
        assert errs[-1] <= 2 * errs[0] + 2 * logit * 2.0 ** -24, errs


@pytest.mark.parametrize("n_q,dim,kv_dtype", [
    (3, 128, "bf16"),                      # 15 columns, logits written
    (6, 64, "f16"),                        # 30 columns, logits written
    (7, 128, "f16"),                       # 35 columns: logits not written
    (9, 64, "bf16"),
])
def test_chunk_queries_may_begin_at_any_element(n_q, dim, kv_dtype):
    """Queries that are contiguous but begin 2, 8 or 16 bytes into an allocation: the same bits as aligned ones."""
    import paper_2605_09490_amd as tkv
    cfg = small_config(name="offset", n_layers=1, batch=2, n_q_heads=10, n_kv_heads=2, head_dim=dim, kv_dtype=kv_dtype,
                       context=333, decode_steps=n_q, k_window=16, sigma=1.0)
    print(f"[case] queries at an offset, chunk of {n_q}, {dim}, {kv_dtype}", flush=True)
    from tkv_synth import Workload
    wl = Workload(cfg, device="cuda")
    k_new, v_new, q = _step_rows(wl, n_q)
    seen = []
    for off in (0, 1, 4, 8):
        kv = tkv.TieredKV(1, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, dim, cfg.max_tokens, kv_dtype=kv_dtype, k_window=16, prefetch_mode="lazy")
        kv.append(0, *wl.context_kv(0))
        kv.append(0, k_new, v_new)
        q_off = torch.empty(q.numel() + 8, dtype=q.dtype, device="cuda")[off:off + q.numel()].view(q.shape)
        assert q_off.copy_(q).data_ptr() % 16 == 2 * off % 16
        seen.append((kv.attend_and_score_chunk(0, q_off).cpu(), kv.get_scores().copy()))
        kv.close()
    for out, scores in seen[1:]:
        assert torch.equal(out, seen[0][0]) and np.array_equal(scores.view(np.uint32), seen[0][1].view(np.uint32))


@pytest.mark.parametrize("heads,kv_heads,dim,kv_dtype", [(8, 2, 64, "bf16"), (7, 1, 64, "f16"), (16, 2, 64, "bf16"), (10, 2, 128, "f16"), (8, 2, 64, "f32")])
def test_single_queries_may_begin_at_any_element(heads, kv_heads, dim, kv_dtype):
    """The same for one query token per sequence, in per-layer calls and in a step over 96 pairs (one workgroup each)."""
    import paper_2605_09490_amd as tkv
    from tkv_synth import Workload
    L = 48 // kv_heads
    cfg = small_config(name="offset", n_layers=L, batch=2, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=dim, kv_dtype=kv_dtype,
                       context=333, decode_steps=2, k_window=16, sigma=1.0)
    print(f"[case] single queries at an offset, {heads}/{kv_heads} heads, {dim}, {kv_dtype}", flush=True)
    wl = Workload(cfg, device="cuda")
    k_all, v_all, q_all = wl.decode_inputs(0, 1)
    q = q_all[0]
    seen = []
    for off in (0, 1, 4, 8):
        kv = tkv.TieredKV(L, cfg.batch, heads, kv_heads, dim, cfg.max_tokens, kv_dtype=kv_dtype, k_window=16, prefetch_mode="lazy")
        for l in range(L):
            kv.append(l, *wl.context_kv(l))
        q_off = torch.empty(q.numel() + 8, dtype=q.dtype, device="cuda")[off:off + q.numel()].view(q.shape)
        q_off.copy_(q)
        step = kv.decode_step(k_all[0], v_all[0], q_off).cpu()
        call = kv.attend_and_score(1, q_off[1]).cpu()
        seen.append((step, call, kv.get_scores().copy()))
        kv.close()
    for step, call, scores in seen[1:]:
        assert torch.equal(step, seen[0][0]) and torch.equal(call, seen[0][1])
        assert np.array_equal(scores.view(np.uint32), seen[0][2].view(np.uint32))


@pytest.mark.parametrize("kv_dtype,t2", [("bf16", "int8_row"), ("f16", "int4_g32")])
def test_whole_pairs_keep_the_precision_of_split_ones(kv_dtype, t2):
    """A workgroup that walks a whole pair adds far more rows into one binary32 sum than a split one does, T2 codes among
    them.  Outputs of a step (one workgroup per pair) against 64 bits, beside those of per-layer calls (32 to 64 workgroups
    per pair) on the same cache.  The rounding of a sum of n like terms grows as the root of n, here by a factor of sqrt(8) and
    only in the part of the error that comes from that sum (a third or less of it): twice the per-layer calls' error."""
    from gpu_common import to_f64
    import paper_2605_09490_amd as tkv
    from oracle import tkv_oracle as O
    from tkv_synth import Workload
    cfg = small_config(name="precision", kv_dtype=kv_dtype, t2_format=t2, k_window=16, sigma=1.0, **PRECISION)
    cfg = dataclasses.replace(cfg, recipe="bias")
    print(f"[case] {kv_dtype} {t2}", flush=True)
    wl = Workload(cfg, device="cuda")
    kv = [tkv.TieredKV(cfg.n_layers, 1, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens, kv_dtype=kv_dtype,
                       t2_format=t2, k_window=16, prefetch_mode="lazy", host_rows=64, staging_rows=64) for _ in range(2)]
    orc = O.OracleCache(2, 1, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens, kv_dtype=kv_dtype, t2_format=t2, k_window=16)
    for l in range(cfg.n_layers):
        k, v = wl.context_kv(l)
        for c in kv:
            c.append(l, k, v)
        if l < 2:
            orc.append(l, to_f64(k), to_f64(v))
    tiers = np.where(np.random.default_rng(5).random((1, cfg.context)) < 0.15, 2, 0).astype(np.uint8)
    tiers[:, :4] = 0
    tiers[:, -16:] = 0
    for c in (*kv, orc):
        c.set_tiers(tiers)
        c.migrate()
    k_all, v_all, q_all = wl.decode_inputs(0, 1)
    step = kv[0].decode_step(k_all[0], v_all[0], q_all[0])
    err = np.zeros((2, 2))
    for l in range(cfg.n_layers):
        kv[1].append(l, k_all[0, l], v_all[0, l])
        call = kv[1].attend_and_score(l, q_all[0, l])
        if l < 2:
            orc.append(l, to_f64(k_all[0, l]), to_f64(v_all[0, l]))
            ref = orc.attend_and_score(l, to_f64(q_all[0, l]))
            err[0, l], err[1, l] = (np.linalg.norm(to_f64(o) - ref) / np.linalg.norm(ref) for o in (step[l], call))
    print(f"[case] error of a step {err[0]}, of per-layer calls {err[1]}", flush=True)
    assert (err[0] <= 2 * err[1]).all(), err
    for c in kv:
        c.close()


def test_many_tiles_per_wave():
    """256 (sequence, kv head) pairs leave two workgroups per pair: every wave walks 8+ tiles of list F and the Q waves
    several of list Q, so the steady-state part of the fetch pipeline (not only its first and last tile) is compared
    element by element."""
    cfg = small_config(name="deep", n_layers=1, batch=32, n_q_heads=8, n_kv_heads=8, head_dim=64, kv_dtype="bf16",
                       context=4200, decode_steps=3, policy_ppm=(300_000, 400_000, 270_000, 30_000), k_window=64)
    _run_shape(cfg, "lazy", steps_before=1, steps_after=1)


def test_batch_above_the_kernel_argument_limit():
    """More than 64 sequences: list lengths and the wave split are read from device counters instead of kernel
    arguments."""
    cfg = small_config(name="wide", n_layers=1, batch=70, n_q_heads=4, n_kv_heads=2, head_dim=64, kv_dtype="f32",
                       context=200, decode_steps=3, policy_ppm=(400_000, 300_000, 250_000, 50_000), k_window=16)
    _run_shape(cfg, "wait", steps_before=1, steps_after=1)


def test_one_sequence_many_splits():
    """A single long sequence with 8 kv heads of 8 query heads each is split 32 ways per kv head: the per-split softmax
    statistics (8 x 32 x 2 x 8 floats) exceed the finishing kernel's LDS copy and are read from memory instead."""
    cfg = small_config(name="solo", n_layers=1, batch=1, n_q_heads=64, n_kv_heads=8, head_dim=64, kv_dtype="bf16",
                       context=9000, decode_steps=3, policy_ppm=(300_000, 400_000, 270_000, 30_000), k_window=64)
    _run_shape(cfg, "wait", steps_before=1, steps_after=1)


def test_14b_full_depth_score_mass():
    """The benchmark's own configuration at full depth (48 layers, batch 8, 4096-token context, lazy prefetch): after
    s decode steps with one re-tiering in between, every sequence's cumulative scores sum to s (Eq. 1 with the scale
    1/(L*Hq): each call adds one unit of probability per query head; evicted positions keep what they had), and an
    evicted position's score does not change any more."""
    import paper_2605_09490_amd as tkv
    from tkv_synth import Workload
    cfg = dataclasses.replace(CONFIGS["14b"], decode_steps=4)
    print(f"[case] 14b full depth L={cfg.n_layers} B={cfg.batch} ctx={cfg.context}", flush=True)
    wl = Workload(cfg, device="cuda")
    gpu = tkv.TieredKV(cfg.n_layers, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.max_tokens,
                       kv_dtype=cfg.kv_dtype, t2_format=cfg.t2_format, k_sink=cfg.k_sink, k_window=cfg.k_window,
                       prefetch_mode="lazy")
    for l in range(cfg.n_layers):
        k, v = wl.context_kv(l)
        gpu.append(l, k, v)
    del k, v
    k_all, v_all, q_all = wl.decode_inputs(0, 4)
    gpu.decode_step(k_all[0], v_all[0], q_all[0])
    gpu.classify(cfg.policy_ppm)
    gpu.migrate()
    n = gpu.layer_length(0)
    tiers = gpu.get_tiers()[:, :n]
    frozen = gpu.get_scores()[:, :n][tiers == 3].copy()
    assert frozen.size > 0
    for s in range(1, 4):
        gpu.decode_step(k_all[s], v_all[s], q_all[s])
    sc = gpu.get_scores().astype(np.float64)
    n2 = gpu.layer_length(0)
    assert np.abs(sc[:, :n2].sum(1) / 4.0 - 1.0).max() < 1e-4
    assert np.array_equal(gpu.get_scores()[:, :n][tiers == 3], frozen)
    st = gpu.get_stats()
    assert st["tier_count"][1] > 0 and st["tier_count"][2] > 0 and st["tier_count"][3] > 0
    gpu.close()


def test_14b_shape_chunk_of_four_query_tokens():
    """Four query tokens per sequence at the 14B per-layer shape (two layers), after one decode step and a
    re-tiering: every query's output and the scores against the oracle; prints the time of the chunk call."""
    from gpu_common import Pair, assert_out_close, assert_scores_close, to_f64
    cfg = dataclasses.replace(CONFIGS["14b"], n_layers=2, decode_steps=5)
    print(f"[case] 14b-shaped chunk L={cfg.n_layers} B={cfg.batch} ctx={cfg.context}", flush=True)
    p = Pair(cfg, prefetch_mode="lazy")
    L, T = cfg.n_layers, 4
    k_all, v_all, q_all = p.wl.decode_inputs(0, 1 + T)
    p.gpu.decode_step(k_all[0], v_all[0], q_all[0])
    for l in range(L):
        p.orc.append(l, to_f64(k_all[0, l]), to_f64(v_all[0, l]))
        p.orc.attend_and_score(l, to_f64(q_all[0, l]))
    n = p.gpu.layer_length(0)
    p.gpu.classify(cfg.policy_ppm)
    plan = p.gpu.get_pending_tiers()[:, :n]
    p.gpu.migrate()
    p.orc.set_tiers(plan); p.orc.migrate()
    p.gpu.wait_prefetch()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for l in range(L):
        k = torch.cat([k_all[1 + j, l] for j in range(T)], dim=1)          # [B, T, Hkv, D]
        v = torch.cat([v_all[1 + j, l] for j in range(T)], dim=1)
        p.append(l, k, v)
    for l in range(L):
        q = torch.stack([q_all[1 + j, l] for j in range(T)], dim=1).contiguous()
        ev0.record()
        out = p.gpu.attend_and_score_chunk(l, q)
        ev1.record()
        ref = p.orc.attend_and_score_chunk(l, to_f64(q))
        torch.cuda.synchronize()
        print(f"[case] layer {l}: chunk of {T} took {ev0.elapsed_time(ev1) * 1e3:.1f} us", flush=True)
        for j in range(T):
            assert_out_close(to_f64(out[:, j]), ref[:, j], cfg.kv_dtype, f"layer {l} query {j}")
    ss = 1.0 / (cfg.n_layers * cfg.n_q_heads)
    assert_scores_close(p.gpu.get_scores(), p.orc.score, n + T, (1 + T) * L * cfg.n_q_heads * ss)
    p.close()


def test_14b_shape_streamed_t1():
    """The 14B per-layer shape with streamed T1 (three layers, so a frame is refilled while the other is read): all
    outputs and scores against the oracle."""
    _run_shape(dataclasses.replace(CONFIGS["14b"], n_layers=3, decode_steps=3), "stream")


def test_batch_above_the_kernel_argument_limit_streamed_t1():
    """More than 64 sequences with streamed T1: the second attention launch and the finishing kernel take the T1
    list's length and its first logits tile from device counters."""
    cfg = small_config(name="wide", n_layers=2, batch=70, n_q_heads=4, n_kv_heads=2, head_dim=64, kv_dtype="bf16",
                       context=200, decode_steps=3, policy_ppm=(400_000, 300_000, 250_000, 50_000), k_window=16)
    _run_shape(cfg, "stream", steps_before=1, steps_after=2)


def test_host_code_under_sanitizers():
    """A randomised sequence of plans, decode steps, store rewrites and inspections in all three prefetch modes, run by a
    build of the host code with AddressSanitizer and UndefinedBehaviorSanitizer (host side only; the kernels are the
    ordinary ones): any host-memory error or undefined arithmetic in the bookkeeping aborts it."""
    import os
    import subprocess
    from paper_2605_09490_amd import build
    assert os.path.exists(build.HOST_CHECK), "build the sanitized host check first: python paper_2605_09490_amd/build.py"
    print(f"[case] {build.HOST_CHECK}", flush=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:protect_shadow_gap=0", UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([build.HOST_CHECK], capture_output=True, text=True, timeout=200, env=env)
    print(r.stdout[-600:], flush=True)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "host sanitizer check passed" in r.stdout
