"""GPU parity of the window recompute pass (App. C.2) against the oracle.

Attention (kara_recompute_attention): every output element against the
oracle's fp64 causal attention over the same bf16 rows, within

    |o_gpu - o_ora| <= u |o_ora| + 5 u sqrt(sum_j p_j^2 (v_j - o_ora)^2) + 2^-16

with u = 2^-8 and p the oracle's softmax weights.  The kernel rounds each
weight to bf16 (relative error up to u, random in sign) before the value
product and normalises by the sum of the same rounded weights, so the
error is sum_j p_j delta_j (v_j - o), whose standard deviation is at most
u/sqrt(3) times the root above; the output store adds u|o|.  One key
dropped or read twice among n moves o by about |v_j - o|/n, several times
the bound at n = 2048 (a CPU test plants exactly that).

Whole pass (kara_recompute_queries): each layer against the oracle's layer
fed the GPU's own fp32 residual stream entering it.  bf16 keeps 8
significant bits, unit roundoff u = 2^-8.  The GPU stores in bf16 the
normalised activations x (error u|x_i|, which reaches q_j through the
product as about u rms(q)), the projected queries (u times the pair the
rotation mixes) and the rotated queries (u|q_j|).  With pn_j the norm of
the rotated pair holding j:

    q:  |q_gpu - q_ora| <= 2u (|q_ora| + pn + 2 rms(q_ora row))

The residual update dh = h_out - h_in passes through five bf16 stores
(attention output, normalised activations, gate, up, their product) and the
attention's own error (above).  Each store adds noise of random sign on
the order of u times its branch's scale, so the error of dh is noise of
about u rms(dh); its largest element over tens of thousands reaches some
4.5 standard deviations.  Elementwise, and for the noise as a whole:

    h:  |dh_gpu - dh_ora| <= 8u (|dh_ora| + rms(dh_ora row))
        rms(dh_gpu - dh_ora) <= 2u rms(dh_ora)      (also for q)

A wrong sign, index, activation or operand order gives errors of order
rms(dh) itself, hundreds of u.
"""
import math

import numpy as np
import pytest

import kara_inputs as ki
from oracle import kara_recompute as rc
from oracle import to_f64

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _setup(n_seqs, window, n_q, n_kv, d, bs, prefix, tail=(0, 8), seed=0):
    cfg = ki.workload("batch8", n_seqs=n_seqs, n_layers=1, window=window, buffer=0, budget=max(1, window // 5),
                      chunk_budget=0, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=d, block_size=bs, prefix=prefix,
                      tail=tail, num_pages=None, pool_slack=0.25, seed=seed)
    geom = ki.make_geometry(cfg)
    p = geom.params()
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed + 100)
    shape = (geom.num_pages, n_kv, bs, d)
    kp = torch.randn(shape, generator=g, device=dev).to(torch.bfloat16)
    vp = torch.randn(shape, generator=g, device=dev).to(torch.bfloat16)
    nt = len(geom.trig)
    q = torch.randn((nt, window, n_q, d), generator=g, device=dev).to(torch.bfloat16)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    return geom, p, q, kp, vp, T(geom.trig), T(geom.block_table), T(geom.seq_lens), T(geom.win_start)


def _oracle_attention(geom, p, q_h, kp_h, vp_h, t, with_spread=False):
    import kara_check as kc
    s = int(geom.trig[t])
    p0 = int(geom.win_start[s])
    W = p["window"]
    to64 = lambda a: to_f64(a, "bf16")
    kr = rc.cache_rows(kp_h, geom.block_table[s], p0 + W, p["block_size"], to64)
    vr = rc.cache_rows(vp_h, geom.block_table[s], p0 + W, p["block_size"], to64)
    qs = to64(q_h[t])
    scale = 1.0 / math.sqrt(p["head_dim"])
    o = rc.causal_window_attention(qs, kr, vr, p0, scale)
    if not with_spread:
        return o
    return o, kc.attention_spread(qs, kr, vr, p0, scale, o)


@pytest.mark.parametrize("window,n_q,n_kv,d,bs,prefix", [
    (64, 8, 2, 128, 16, (0, 0)),           # no prefix: token 0 sees only itself
    (200, 8, 2, 128, 16, (0, 300)),        # window not a multiple of a chunk, ragged prefix
    (96, 40, 8, 128, 7, (10, 130)),        # G = 5 (Qwen3-14B), unaligned blocks
    (128, 4, 4, 64, 16, (0, 100)),         # G = 1, d = 64
    (256, 32, 8, 128, 256, (0, 600)),      # serving geometry: 256-token blocks
    (64, 8, 2, 128, 1, (2050, 2400)),      # one-token blocks past 2048: a second block-table segment
    (80, 8, 2, 64, 2, (4050, 4500)),       # d = 64, two-token blocks past 4096: the same switch
])
def test_attention_parity(window, n_q, n_kv, d, bs, prefix):
    from paper_2607_01237_amd import kara
    _need_gpu()
    print(f"\n[case] recompute attention W={window} {n_q}/{n_kv} d={d} bs={bs} prefix={prefix}", flush=True)
    geom, p, q, kp, vp, trig, bt, lens, ws = _setup(3, window, n_q, n_kv, d, bs, prefix)
    params = kara.make_params(p, geom.block_table.shape[0])
    out = torch.full_like(q, float("nan"))
    status = torch.full((len(geom.trig),), -7, dtype=torch.int32, device=q.device)
    kara.recompute_attention(params, trig, q, kp, vp, bt, lens, ws, out, status)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    got = to_f64(ki.raw_numpy(out), "bf16")
    q_h, kp_h, vp_h = ki.raw_numpy(q), ki.raw_numpy(kp), ki.raw_numpy(vp)
    import kara_check as kc
    worst = 0.0
    for t in range(len(geom.trig)):
        want, spread = _oracle_attention(geom, p, q_h, kp_h, vp_h, t, with_spread=True)
        worst = max(worst, kc.check_attention(got[t], want, spread, f"trigger {t}"))
    print(f"[case] ok, max abs err {worst:.2e}", flush=True)


@pytest.mark.parametrize("n_seqs,window,n_q,n_kv,d", [
    (1, 129, 4, 1, 128),      # one unit: eight pieces, most of them empty; 128-row workgroups
    (5, 70, 6, 2, 64),        # ten units: four pieces each; ranks by length
    (7, 280, 16, 4, 128),     # 28 units: two pieces, 128-row workgroups on 252 of 256 CUs ...
    (7, 280, 20, 5, 128),     # ... and 256-row workgroups past them (35 units, eight pieces)
    (3, 600, 32, 8, 128),     # 24 units: whole units, an uneven last row block
])
def test_attention_block_dealing(n_seqs, window, n_q, n_kv, d):
    # every row block of every unit is computed once, whatever the pieces and
    # the rank order: the parity bound of the file header, all sequences
    import kara_check as kc
    from paper_2607_01237_amd import kara
    _need_gpu()
    print(f"\n[case] attention dealing {n_seqs} x W={window} {n_q}/{n_kv} d={d}", flush=True)
    geom, p, q, kp, vp, trig, bt, lens, ws = _setup(n_seqs, window, n_q, n_kv, d, 16, (0, 400), seed=3)
    params = kara.make_params(p, geom.block_table.shape[0])
    trig = trig.flip(0).contiguous()
    out = torch.full_like(q, float("nan"))
    status = torch.full((n_seqs,), -7, dtype=torch.int32, device=q.device)
    kara.recompute_attention(params, trig, q, kp, vp, bt, lens, ws, out, status)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    geom.trig = geom.trig[::-1].copy()
    got = to_f64(ki.raw_numpy(out), "bf16")
    q_h, kp_h, vp_h = ki.raw_numpy(q), ki.raw_numpy(kp), ki.raw_numpy(vp)
    for t in range(n_seqs):
        want, spread = _oracle_attention(geom, p, q_h, kp_h, vp_h, t, with_spread=True)
        kc.check_attention(got[t], want, spread, f"trigger {t}")
    print("[case] ok", flush=True)


def test_attention_flags_bad_windows():
    from paper_2607_01237_amd import kara
    _need_gpu()
    print("\n[case] recompute attention status flags", flush=True)
    geom, p, q, kp, vp, trig, bt, lens, ws = _setup(3, 64, 8, 2, 128, 16, (0, 50))
    params = kara.make_params(p, geom.block_table.shape[0])
    bad_ws = ws.clone()
    s1 = int(geom.trig[1])
    bad_ws[s1] = int(geom.seq_lens[s1]) - 10          # window runs past the end
    trig2 = trig.clone()
    trig2[2] = trig2[0]                                # listed twice
    out = torch.zeros_like(q)
    status = torch.full((len(geom.trig),), -7, dtype=torch.int32, device=q.device)
    kara.recompute_attention(params, trig2, q, kp, vp, bt, lens, bad_ws, out, status)
    torch.cuda.synchronize()
    st = status.cpu().numpy()
    assert st[1] == kara.SEQ_BAD_WINDOW
    assert st[0] & kara.SEQ_DUP_TRIGGER and st[2] & kara.SEQ_DUP_TRIGGER
    assert (out[1].float() == 0).all() and (out[2].float() == 0).all()


def _weights(rng_t, L, D, F, HD, dev):
    def w(shape, fan_in):
        return (torch.randn(shape, generator=rng_t, device=dev) / math.sqrt(fan_in)).to(torch.bfloat16)
    out = []
    for _ in range(L):
        out.append(dict(w_q=w((D, HD), D), w_o=w((HD, D), HD), w_gate=w((D, F), D), w_up=w((D, F), D),
                        w_down=w((F, D), F),
                        g_attn=(1.0 + 0.1 * torch.randn(D, generator=rng_t, device=dev)).to(torch.bfloat16),
                        g_ffn=(1.0 + 0.1 * torch.randn(D, generator=rng_t, device=dev)).to(torch.bfloat16)))
    return out


def _f64(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("window,n_q,n_kv,d,D,F,bs", [
    (64, 8, 2, 128, 512, 1024, 16),
    (80, 10, 2, 64, 384, 768, 7),
])
def test_recompute_pass_layers(window, n_q, n_kv, d, D, F, bs):
    from paper_2607_01237_amd import kara
    _need_gpu()
    L = 2
    print(f"\n[case] recompute pass W={window} {n_q}/{n_kv} d={d} D={D} F={F} bs={bs}", flush=True)
    geom, p, _, kp0, vp0, trig, bt, lens, ws = _setup(3, window, n_q, n_kv, d, bs, (0, 200), seed=1)
    dev = kp0.device
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    kp = [kp0] + [torch.randn_like(kp0, dtype=torch.float32).to(torch.bfloat16) for _ in range(L - 1)]
    vp = [vp0] + [torch.randn_like(vp0, dtype=torch.float32).to(torch.bfloat16) for _ in range(L - 1)]
    wts = _weights(g, L, D, F, n_q * d, dev)
    nt = len(geom.trig)
    h0 = torch.randn((nt, window, D), generator=g, device=dev)
    rope_pos0 = (torch.from_numpy(geom.win_start).to(dev) + 5000).to(torch.int32)   # positions after compressions
    params = kara.make_params(p, geom.block_table.shape[0])
    model = kara.make_model(D, F, rope_theta=1e6, rms_eps=1e-6)
    wsp = torch.empty(kara.recompute_workspace_size(params, model, nt), dtype=torch.uint8, device=dev)
    status = torch.full((nt,), -7, dtype=torch.int32, device=dev)

    # layer by layer, each from the GPU's own residual stream
    h = h0.clone()
    q_layers = []
    for l in range(L):
        h_next = torch.empty_like(h)
        q = torch.empty((1, nt, window, n_q, d), dtype=torch.bfloat16, device=dev)
        kara.recompute_queries(params, model, trig, [wts[l]], h, h_next, [kp[l]], [vp[l]], bt, lens, ws, rope_pos0,
                               q, status, wsp)
        torch.cuda.synchronize()
        assert (status.cpu().numpy() == 0).all()
        wt64 = {k_: _f64(v_) for k_, v_ in wts[l].items()}
        dims = dict(n_q_heads=n_q, head_dim=d, rms_eps=1e-6, rope_theta=1e6, block_size=bs)
        to64 = lambda a: to_f64(a, "bf16")
        kh, vh = ki.raw_numpy(kp[l]), ki.raw_numpy(vp[l])
        for t in range(nt):
            s = int(geom.trig[t])
            p0 = int(geom.win_start[s])
            kr = rc.cache_rows(kh, geom.block_table[s], p0 + window, bs, to64)
            vr = rc.cache_rows(vh, geom.block_table[s], p0 + window, bs, to64)
            hin = _f64(h[t])
            q_ora, h_ora, _ = rc.recompute_layer(hin, wt64, kr, vr, p0, p0 + 5000, dims)
            q_gpu = to_f64(ki.raw_numpy(q[0, t]), "bf16")
            rms = np.sqrt((q_ora ** 2).mean(axis=-1, keepdims=True))
            half = d // 2
            pn = np.sqrt(q_ora[..., :half] ** 2 + q_ora[..., half:] ** 2)
            pn = np.concatenate([pn, pn], axis=-1)
            err = np.abs(q_gpu - q_ora)
            ratio_q = float((err / (np.abs(q_ora) + pn + 2 * rms)).max()) / 2.0 ** -8
            dh_ora = h_ora - hin
            dh_gpu = _f64(h_next[t]) - hin
            rms_h = np.sqrt((dh_ora ** 2).mean(axis=-1, keepdims=True))
            err_h = np.abs(dh_gpu - dh_ora)
            ratio_h = float((err_h / (np.abs(dh_ora) + rms_h)).max()) / 2.0 ** -8
            noise_q = float(np.sqrt((err ** 2).mean() / (q_ora ** 2).mean())) / 2.0 ** -8
            noise_h = float(np.sqrt((err_h ** 2).mean() / (dh_ora ** 2).mean())) / 2.0 ** -8
            print(f"[case] layer {l} trigger {t}: q err {err.max():.3e} ({ratio_q:.2f} of 2 u), noise {noise_q:.2f} u; "
                  f"dh err {err_h.max():.3e} ({ratio_h:.2f} of 8 u), noise {noise_h:.2f} u", flush=True)
            assert ratio_q <= 2.0, f"layer {l} trigger {t}: q max err {err.max():.3e}"
            assert ratio_h <= 8.0, f"layer {l} trigger {t}: h max err {err_h.max():.3e}"
            assert noise_q <= 2.0 and noise_h <= 2.0, (noise_q, noise_h)
        q_layers.append(q[0].clone())
        h = h_next

    # one call over both layers gives the same bits as the layer-by-layer calls
    q_all = torch.empty((L, nt, window, n_q, d), dtype=torch.bfloat16, device=dev)
    h_all = torch.empty_like(h0)
    kara.recompute_queries(params, model, trig, wts, h0, h_all, kp, vp, bt, lens, ws, rope_pos0, q_all, status, wsp)
    torch.cuda.synchronize()
    for l in range(L):
        assert torch.equal(q_all[l].view(torch.int16), q_layers[l].view(torch.int16)), f"layer {l} queries"
    assert torch.equal(h_all, h)
    # in place (hidden_out is hidden_in), with scratch full of ones so that a
    # product run ahead of its inputs would show: the same bits
    h_inout = h0.clone()
    wsp.view(torch.bfloat16)[:wsp.numel() // 2].fill_(1.0)
    kara.recompute_queries(params, model, trig, wts, h_inout, h_inout, kp, vp, bt, lens, ws, rope_pos0, q_all, status,
                           wsp)
    torch.cuda.synchronize()
    assert torch.equal(h_inout, h) and torch.equal(q_all[L - 1].view(torch.int16), q_layers[L - 1].view(torch.int16))
    # after the first call on the device, calls allocate nothing: the device's
    # free memory is unchanged across another full call
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    kara.recompute_queries(params, model, trig, wts, h0, h_all, kp, vp, bt, lens, ws, rope_pos0, q_all, status, wsp)
    torch.cuda.synchronize()
    free1, _ = torch.cuda.mem_get_info()
    assert free1 == free0, f"a recompute call took {free0 - free1} bytes of device memory"
    print("[case] ok", flush=True)


def test_recompute_then_compress():
    """The event pipeline: the recompute pass writes the scoring queries of
    every layer, kara_compress_window consumes them, and the result passes
    P1-P4 against the oracle run on the same queries (the layouts of the
    two entry points agree)."""
    import kara_check as kc
    from paper_2607_01237_amd import kara
    _need_gpu()
    print("\n[case] recompute -> compress", flush=True)
    c = kc.setup(ki.workload("batch8", n_seqs=3, n_layers=2, window=128, budget=26, n_q_heads=8, n_kv_heads=2,
                             prefix=(10, 100), tail=(0, 8), num_pages=None, pool_slack=0.25))
    p = c.p
    L, nt = len(c.kp), c.trig.numel()
    W, Hq, d = p["window"], p["n_q_heads"], p["head_dim"]
    D, F = 256, 512
    dev = c.q.device
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    wts = _weights(g, L, D, F, Hq * d, dev)
    model = kara.make_model(D, F, rope_theta=1e6, rms_eps=1e-6)
    h0 = torch.randn((nt, W, D), generator=g, device=dev)
    h1 = torch.empty_like(h0)
    q = torch.empty((L, nt, W, Hq, d), dtype=torch.bfloat16, device=dev)
    status = torch.full((nt,), -7, dtype=torch.int32, device=dev)
    wsp = torch.empty(kara.recompute_workspace_size(c.params, model, nt), dtype=torch.uint8, device=dev)
    kara.recompute_queries(c.params, model, c.trig, wts, h0, h1, c.kp, c.vp, c.bt, c.seq_lens, c.win_start,
                           c.win_start, q, status, wsp)
    torch.cuda.synchronize()
    assert (status.cpu().numpy() == 0).all()
    assert torch.isfinite(q.float()).all()
    c.q = q
    c.host["q"] = ki.raw_numpy(q)
    rep, _ = kc.full_check(c)
    print(f"[case] ok {rep}", flush=True)
