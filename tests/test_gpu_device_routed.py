"""Layers whose experts all hold a slot follow the routing on the device; the
host decides only where an expert may have to be loaded.  Both must give the
same routing and the same output bits, whatever slots the experts hold and
whenever a layer changes from one to the other."""
import numpy as np
import pytest

import oracle as o
import workload as w
from paper_2607_24787_amd import spp
from workload import gen

pytestmark = pytest.mark.gpu

BASE = w.MoEConfig(name="routed_bf16_D640_n40_k5", L=4, D=640, n=40, K=5, I=100, r=12, S=11, windows=(2,), tokens=8,
                   seed=41)


@pytest.mark.parametrize("cfg", [
    BASE,                                                  # workgroup-wide router tail (r = 12)
    BASE.with_(r=16, n_shared=1),                          # single-wave tail, one expert per lane
    BASE.with_(r=16, n=100, K=6, has_proj=True),           # two experts per lane, projection in front
    BASE.with_(D=256, I=96, r=8, codec="q4"),
    # router and FFN in one launch: rows past 2,048 columns, exact and ragged, every adapter width and list
    BASE.with_(D=2304, I=64, r=8, n=16, S=9, codec="q4"),
    BASE.with_(D=4096, I=33, r=64, n=16, S=9, codec="q4", n_shared=2),
    BASE.with_(D=2056, I=61, r=64, n=128, K=8, S=20),
    BASE.with_(D=4096, I=5, r=8, n=9, K=1, S=3),
    BASE.with_(D=1300, I=37, r=8, dtype="f32", K=3, n_shared=1, has_proj=True),
    BASE.with_(D=128, I=64, r=8, dtype="f32", batch=3, S=17, n_shared=1),
    BASE.with_(I=100, batch=3, S=17),                      # bf16 in the unit layout (I not a multiple of 16)
], ids=["b1_wide_tail", "b1_one_wave", "b1_n100_proj", "q4", "q4_ragged", "q4_long", "b1_long_ragged", "b1_k1", "b1_f32",
        "f32_b3", "bf16_units_b3"])
def test_device_and_host_routed_layers_give_the_same_bits(cfg):
    from paper_2607_24787_amd.model import OffloadedMoEStack
    h0 = gen.hidden_states(cfg, tokens=cfg.tokens)
    host = OffloadedMoEStack(cfg)                # S < n: every layer decided on the host
    full = OffloadedMoEStack(cfg, S=cfg.n)       # every expert resident
    try:
        table = np.random.default_rng(5).permutation(cfg.n).astype(np.int32)
        part = table.copy()
        part[1::3] = -1
        for l in range(cfg.L):
            spp.spp_set_slot_table(full.ctx, l, table, np.zeros(cfg.n, np.int64))
        for t in range(cfg.tokens):
            if t == 3:  # two layers lose a third of their experts and load them back as they are needed
                for l in (1, 2):
                    spp.spp_set_slot_table(full.ctx, l, part, np.zeros(cfg.n, np.int64))
            if t == 6:  # other slots than before
                spp.spp_set_slot_table(full.ctx, 1, table[::-1].copy(), np.zeros(cfg.n, np.int64))
            before = _paths(full)
            ref = host.decode_step_from(_in(host, h0[t]), 2)
            got = full.decode_step_from(_in(full, h0[t]), 2)
            routed, one = (a - b for a, b in zip(_paths(full), before))
            if t < 3:
                assert routed == cfg.L and one == sum(_one_launch(cfg, l) for l in range(cfg.L))
            elif t == 3:
                assert routed == cfg.L - 2
            for l in range(cfg.L):
                assert np.array_equal(got[l][0], ref[l][0]), (t, l)
                assert np.array_equal(got[l][1], ref[l][1]), (t, l)
                distinct = len(set(got[l][0].ravel().tolist()))
                assert got[l][2].ready_on_time + got[l][2].waited == distinct, (t, l)
                if t < 3:
                    assert got[l][2].hits == distinct and got[l][2].misses == 0 and got[l][2].prefetched == 0
            assert np.array_equal(full.download(full.hbuf[0]), host.download(host.hbuf[0])), t
        assert spp.spp_get_clock(full.ctx) == cfg.tokens * cfg.L
        assert _paths(host) == (0, 0)
        _, stamps = spp.spp_get_slot_table(full.ctx, 0, cfg.n)
        last = set(got[0][0].ravel().tolist())
        assert [int(s) == (cfg.tokens - 1) * cfg.L + 1 for s in stamps] == [int(e) in last for e in table]
    finally:
        host.close()
        full.close()


def _paths(st):
    return spp.spp_debug_get_paths(st.ctx)


def _one_launch(cfg, l):
    """Whether a resident layer's router and FFN go out as one launch."""
    adapter = l < cfg.L - 1 and cfg.r > 0
    return cfg.batch == 1 and cfg.n <= 128 and (not adapter or (cfg.dtype == "bf16" and cfg.r <= 64 and cfg.r % 8 == 0))


ONE_LAUNCH = [
    BASE.with_(r=16, n_shared=1),
    BASE.with_(r=16, n=100, K=6, has_proj=True),
    BASE.with_(D=256, I=96, r=8, codec="q4"),
    BASE.with_(D=4096, I=33, r=64, n=16, K=2, codec="q4", n_shared=2, has_proj=True),
    BASE.with_(D=2056, I=61, r=64, n=128, K=8),
    BASE.with_(D=4096, I=5, r=8, n=9, K=1),
    BASE.with_(D=1300, I=37, r=8, dtype="f32", K=3, n_shared=1),
]


@pytest.mark.parametrize("cfg", ONE_LAUNCH, ids=["n40", "n100_proj", "q4", "q4_long_proj", "long_ragged", "k1", "f32"])
def test_ffn_workgroups_that_do_not_see_the_routing_form_it(cfg):
    """A launch's FFN workgroups must not depend on its router's being on the device, nor the tail of an adapter-only
    launch on its rows': with no polls every one of them forms the routing (the hidden units) itself, and with one poll
    some do.  Same bits."""
    from paper_2607_24787_amd.model import OffloadedMoEStack
    st = OffloadedMoEStack(cfg, S=cfg.n)
    h0 = gen.hidden_states(cfg, tokens=4)
    x = st.torch.randn(cfg.D, device=st.device, generator=st.torch.Generator(st.device).manual_seed(3))
    runs = []
    one = sum(_one_launch(cfg, l) for l in range(cfg.L))
    try:
        for polls in (-1, 0, 1):
            print(f"[route polls] {cfg.D} {cfg.codec} {cfg.dtype} polls={polls}", flush=True)
            spp.spp_debug_set_self_polls(st.ctx, polls)
            spp.spp_reset_run_stats(st.ctx)
            st.reset()
            runs.append([])
            for t in range(4):
                out = st.decode_step_from(_in(st, h0[t]), 0)
                runs[-1] += [a for l in out for a in l[:2]] + [st.download(st.hbuf[0])]
                runs[-1].append(spp.adapter_predict(st.ctx, 0, x.data_ptr(), 1, cfg.n))
            assert _paths(st) == (4 * cfg.L, 4 * one)
    finally:
        st.close()
    for other in runs[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(runs[0], other))


def test_two_contexts_decode_on_two_streams():
    """Two contexts that fill the device from two threads, each on a stream of its own: what each gives alone."""
    import threading

    import torch
    from paper_2607_24787_amd.model import OffloadedMoEStack
    cfg = w.MoEConfig(name="two_streams", L=6, D=1280, n=64, K=6, I=896, r=32, S=64, windows=(1,), tokens=24, n_shared=2,
                      expert_layers=1, seed=53)
    h0 = gen.hidden_states(cfg, tokens=cfg.tokens)
    torch.cuda.set_device(0)
    stacks = []
    for _ in range(2):
        with torch.cuda.stream(torch.cuda.Stream()):
            stacks.append(OffloadedMoEStack(cfg))
    h_in = [[torch.from_numpy(h.reshape(-1).view(np.uint8).copy()).to("cuda:0") for h in h0] for _ in stacks]
    outs = [[torch.empty_like(h) for h in hs] for hs in h_in]
    errors = []

    def run(k):
        try:
            st = stacks[k]
            for h, out in zip(h_in[k], outs[k]):
                spp.spp_decode_step(st.ctx, cfg.L, h.data_ptr(), out.data_ptr(), st.hbuf[1].data_ptr(), 1, cfg.K, 1)
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    try:
        torch.cuda.synchronize()
        run(0)
        torch.cuda.synchronize()
        want = [out.clone() for out in outs[0]]
        for rep in range(4):
            print(f"[two streams] pass {rep}", flush=True)
            for o_ in outs:
                for out in o_:
                    out.zero_()
            torch.cuda.synchronize()
            threads = [threading.Thread(target=run, args=(k,)) for k in range(2)]
            for th in threads:
                th.start()
            for th in threads:
                th.join()
            torch.cuda.synchronize()
            assert not errors, errors
            for k in range(2):
                assert all(torch.equal(a, b) for a, b in zip(outs[k], want)), (rep, k)
    finally:
        for st in stacks:
            st.close()


def _in(st, h):
    """A device copy of stored hidden states that outlives the step."""
    st.h_in = st.torch.from_numpy(np.ascontiguousarray(h).reshape(-1).view(np.uint8).copy()).to(st.device)
    return st.h_in.data_ptr()


# batched: groups of more than 16 and of more than 32 tokens, shared experts over several chunks of tokens, unit
# ranges that end in half a step of 32 units, ranges wide enough for workgroups of 8 waves, more experts than lanes
GROUPED = w.MoEConfig(name="grouped_bf16_D512_n6_k2_I400", L=2, D=512, n=6, K=2, I=400, r=8, S=6, windows=(1,),
                      tokens=2, batch=40, n_shared=1, seed=43)


GROUPED_CFGS = {
    "chunks": GROUPED,
    "wide_ranges": GROUPED.with_(n=4, K=1, I=1104, n_shared=2, batch=75),
    "n140": GROUPED.with_(n=140, K=3, I=784, D=256, n_shared=0, batch=90, r=16),
    "one_tile": GROUPED.with_(n=24, K=5, I=16, D=768, batch=3, has_proj=True),
    "k_eq_n": GROUPED.with_(n=9, K=9, I=336, D=1280, batch=2),
    # the unit layout: several 32-token chunks, one unit past whole workgroups, every chunk count and its tail
    "units_bf16": GROUPED.with_(I=49, D=272, batch=45),
    "units_bf16_full": GROUPED.with_(I=25, D=2048, batch=3, n=12),
    "units_bf16_long": GROUPED.with_(I=9, D=3104, batch=5, n_shared=0),
    "units_f32": GROUPED.with_(I=61, D=1024, dtype="f32", batch=6),
    "units_f32_long": GROUPED.with_(I=30, D=1296, dtype="f32", batch=40, has_proj=True),
}


def _fits_in_rounds(cfg):
    """The tiled layout, and the unit layout where half the experts hold a batch's demand."""
    tiled = cfg.dtype == "bf16" and cfg.D % 256 == 0 and cfg.I % 16 == 0
    return tiled or cfg.K * cfg.batch < cfg.n


@pytest.mark.parametrize("cfg,resident",
                         [pytest.param(c, True, id=f"resident-{k}") for k, c in GROUPED_CFGS.items()]
                         + [pytest.param(c, False, id=f"rounds-{k}") for k, c in GROUPED_CFGS.items() if _fits_in_rounds(c)])
def test_grouped_layers_against_the_oracle(cfg, resident):
    from lockstep import run_lockstep
    from paper_2607_24787_amd.model import OffloadedMoEStack
    st = OffloadedMoEStack(cfg, S=cfg.n if resident else max(cfg.n // 2, 1))
    try:
        rep = run_lockstep(st, cfg, cfg.tokens, 1)
    finally:
        st.close()
    assert rep.max_ulp_h <= 1.0 + 1e-9 and rep.max_err_g <= 1e-5
    assert len(rep.exempt) <= 1


@pytest.mark.parametrize("cfg", [
    GROUPED.with_(n=140, K=3, I=48, batch=7, r=0, S=140),
    GROUPED.with_(n=140, K=3, I=25, batch=3, r=0, S=140, dtype="f32", D=272),
], ids=["tiled", "units_f32"])
def test_batched_selection_without_an_adapter(cfg):
    """The workgroup-wide selection (more than 128 experts) of a full batch where a row of the logit buffer holds
    nothing behind its n logits: its last row ends the buffer."""
    from lockstep import run_lockstep
    from paper_2607_24787_amd.model import OffloadedMoEStack
    st = OffloadedMoEStack(cfg)
    try:
        rep = run_lockstep(st, cfg, cfg.tokens, -1)
    finally:
        st.close()
    assert rep.max_ulp_h <= 1.0 + 1e-9 and rep.max_err_g <= 1e-5
    assert len(rep.exempt) <= 1


@pytest.mark.parametrize("cfg,per_token", [
    (GROUPED.with_(D=2064, n=24, K=8, I=200, batch=2, n_shared=1, S=20), True),
    (GROUPED.with_(D=2064, n=48, K=8, I=400, batch=3, n_shared=0, S=30), True),
    (GROUPED.with_(D=1040, n=24, K=8, I=400, batch=2, n_shared=0, S=20, dtype="f32", has_proj=True), True),
    (GROUPED.with_(D=2064, n=140, K=8, I=200, batch=2, n_shared=0, S=20, tokens=1), True),   # workgroup-wide selection
    (GROUPED.with_(D=528, n=24, K=4, I=70, batch=2, n_shared=0, S=20), False),
    (GROUPED.with_(D=3104, n=24, K=3, I=41, batch=5, n_shared=0, S=20), False),   # one row of x at a time
    (GROUPED.with_(D=2048, n=24, K=3, I=41, batch=7, n_shared=1, S=23, dtype="f32"), False),
], ids=["b2", "b3", "f32_b2", "b2_n140", "batched_b2", "batched_long", "batched_f32_long"])
def test_few_tokens_in_the_unit_layout(cfg, per_token):
    """A launch per token or one for the batch: both against the oracle, with the same bits whether the layers are
    resident, decided on the host or timed."""
    from lockstep import run_lockstep
    from paper_2607_24787_amd.model import OffloadedMoEStack
    h0 = gen.hidden_states(cfg, tokens=cfg.tokens)
    outs = []
    for S in (cfg.n, cfg.S):
        st = OffloadedMoEStack(cfg, S=S)
        try:
            rep = run_lockstep(st, cfg, cfg.tokens, 1)
            assert rep.max_ulp_h <= 1.0 + 1e-9 and rep.max_err_g <= 1e-5 and len(rep.exempt) <= 1
            for timing in (0, 1):
                st.reset()
                spp.spp_set_timing(st.ctx, timing)
                spp.spp_reset_run_stats(st.ctx)
                for t in range(cfg.tokens):
                    st.decode_step_from(_in(st, h0[t]), 1)
                    outs.append(st.download(st.hbuf[0]))
                stats = spp.spp_get_run_stats(st.ctx)
                assert stats.ffn_launches == cfg.tokens * cfg.L * (cfg.batch if per_token else 1)
                assert _paths(st)[1] == 0 and (stats.ffn_us > 0) == bool(timing)
        finally:
            st.close()
    for k, out in enumerate(outs):
        assert np.array_equal(out, outs[k % cfg.tokens])


@pytest.mark.parametrize("cfg", [
    GROUPED.with_(I=49, D=272, batch=11),
    GROUPED.with_(I=30, D=1296, dtype="f32", batch=40, has_proj=True, n_shared=2),
], ids=["bf16", "f32_proj"])
def test_unit_layout_batches_in_several_launches(cfg):
    """A batch whose partial rows exceed the buffer goes out in runs of tokens, the last one shorter: the bits of one
    launch, resident and decided on the host (every expert but one resident)."""
    from paper_2607_24787_amd.model import OffloadedMoEStack
    h0 = gen.hidden_states(cfg, tokens=2)
    outs = []
    for S, spare in ((cfg.n, 0), (cfg.n, 1)):
        st = OffloadedMoEStack(cfg, S=S, resident=range(cfg.n - spare))
        try:
            for run in (cfg.batch, 4, 7, 1):
                spp.spp_debug_set_batch_tokens(st.ctx, run)
                st.reset()
                spp.spp_reset_run_stats(st.ctx)
                st.decode_step_from(_in(st, h0[0]), -1)
                outs.append(st.download(st.hbuf[0]))
                assert spp.spp_get_run_stats(st.ctx).ffn_launches == cfg.L * -(-cfg.batch // run)
                assert (_paths(st)[0] == 0) == bool(spare)
            for bad in (0, cfg.batch + 1):
                with pytest.raises(spp.SppError) as e:
                    spp.spp_debug_set_batch_tokens(st.ctx, bad)
                assert e.value.status == spp.SPP_EINVAL
        finally:
            st.close()
    assert all(np.array_equal(out, outs[0]) for out in outs)


def test_grouped_layers_give_the_same_bits_whatever_is_resident():
    from paper_2607_24787_amd.model import OffloadedMoEStack
    cfg = GROUPED.with_(n=24, K=4, I=208, batch=21, n_shared=0)
    h0 = gen.hidden_states(cfg, tokens=2)
    outs = []
    for S in (24, 13, 5):
        st = OffloadedMoEStack(cfg, S=S)
        try:
            outs.append([])
            for t in range(2):
                st.decode_step_from(_in(st, h0[t]), 1)
                outs[-1].append(st.download(st.hbuf[0]))
        finally:
            st.close()
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("cfg", [
    GROUPED.with_(L=2, batch=37),
    GROUPED.with_(L=2, D=272, I=49, batch=6),
    GROUPED.with_(L=2, D=1040, I=61, batch=5, dtype="f32", n_shared=0),
    GROUPED.with_(L=2, D=2064, n=24, K=8, I=200, batch=2),
], ids=["tiled", "units", "units_f32", "token_launches"])
@pytest.mark.parametrize("bad", [np.nan, np.inf], ids=["nan", "inf"])
def test_a_non_finite_token_leaves_the_others_alone(cfg, bad):
    """Every other token of the batch keeps its routing and bits; the call returns, the bad token's output is a NaN."""
    from paper_2607_24787_amd.model import OffloadedMoEStack
    h = gen.hidden_states(cfg, tokens=1)[0].copy()
    b = cfg.batch // 2
    plain = h.copy()
    h[b, 3] = gen.f32_to_bf16_bits(np.float32([bad]))[0] if cfg.dtype == "bf16" else bad
    st = OffloadedMoEStack(cfg, S=cfg.n)
    try:
        runs = []
        for x in (plain, h):
            out = st.decode_step_from(_in(st, x), 0)
            runs.append(([np.delete(l[0], b, 0) for l in out], o.decode(st.download(st.hbuf[0]), cfg.dtype)))
        assert all(np.array_equal(p, q) for p, q in zip(runs[0][0], runs[1][0]))
        assert np.array_equal(np.delete(runs[0][1], b, 0), np.delete(runs[1][1], b, 0))
        assert np.isnan(runs[1][1][b]).all()
    finally:
        st.close()


@pytest.mark.parametrize("I", [80, 400], ids=["one_range", "ranges"])
def test_grouped_layers_with_non_finite_down_weights(monkeypatch, I):
    """An infinite down weight gives the infinity of h's sign (h has 24 significant bits, of which the products take 8
    at a time: a part that is 0 must not turn the output into a NaN), a NaN weight a NaN, and every other output the
    bits it has with zeros in those places."""
    from paper_2607_24787_amd.model import OffloadedMoEStack
    cfg = GROUPED.with_(L=1, I=I)
    per = 60                                       # columns of each expert with an infinite weight, and one with a NaN
    n_all = cfg.n + cfg.n_shared
    cols = np.random.default_rng(7).permutation(cfg.D)[:n_all * (per + 1)].reshape(n_all, per + 1)
    units = np.random.default_rng(8).integers(0, I, size=(n_all, per + 1))
    routed, shared = gen.expert_weights, gen.shared_expert_weights

    def planted(bits):
        def put(ws, e):
            g, u, d = ws
            d = d.copy()
            d[cols[e, :per], units[e, :per]] = bits[0]
            d[cols[e, per], units[e, per]] = bits[1]
            return g, u, d
        monkeypatch.setattr(gen, "expert_weights", lambda c, l, e: put(routed(c, l, e), e))
        monkeypatch.setattr(gen, "shared_expert_weights", lambda c, l, j: put(shared(c, l, j), cfg.n + j))

    h0 = gen.hidden_states(cfg, tokens=1)
    outs = []
    for bits in ((0x7f80, 0x7fc0), (0, 0)):
        planted(bits)
        st = OffloadedMoEStack(cfg)
        try:
            topk = st.decode_step_from(_in(st, h0[0]), -1)[0][0]
            outs.append(o.decode(st.download(st.hbuf[0]), cfg.dtype))
            x = spp.spp_get_last_router_input(st.ctx, cfg.batch, cfg.D).astype(np.float64)
        finally:
            st.close()
    got, plain = outs
    want = plain.copy()
    for e in range(n_all):
        g, u, _ = routed(cfg, 0, e) if e < cfg.n else shared(cfg, 0, e - cfg.n)
        g, u = o.decode(g, cfg.dtype), o.decode(u, cfg.dtype)
        for b in range(cfg.batch):
            if e < cfg.n and e not in topk[b]:
                continue
            a = x[b] @ g.T.astype(np.float64)
            h = a / (1 + np.exp(-a)) * (x[b] @ u.T.astype(np.float64))
            want[b, cols[e, :per]] = np.copysign(np.inf, h[units[e, :per]])
            want[b, cols[e, per]] = np.nan
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("D,I,dtype", [(512, 2600, "bf16"), (640, 2300, "bf16"), (1536, 1801, "bf16"),
                                       (2048, 1900, "bf16"), (2304, 600, "bf16"), (2048, 351, "f32"), (520, 61, "bf16")],
                         ids=["D512", "D640", "D1536", "D2048", "D2304", "f32_D2048", "D520"])
def test_sweep_rounds_of_the_batch_1_ffn(D, I, dtype):
    """Every number of sweep rounds the unit counts lead to, with rows that end inside a wave's chunks."""
    from lockstep import run_lockstep
    from paper_2607_24787_amd.model import OffloadedMoEStack
    cfg = w.MoEConfig(name=f"rounds_D{D}_I{I}", L=1, D=D, n=6, K=4, I=I, r=0, S=6, windows=(1,), tokens=2, dtype=dtype,
                      seed=47)
    st = OffloadedMoEStack(cfg)
    try:
        rep = run_lockstep(st, cfg, cfg.tokens, -1)
    finally:
        st.close()
    assert rep.max_ulp_h <= 1.0 + 1e-9 and not rep.exempt
