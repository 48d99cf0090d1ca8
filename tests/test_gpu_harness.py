"""The decoding-side helpers (include/kara_harness.h) against plain CPU
references: token append into the paged cache (bit-exact rows, lengths and
status bits) and decode attention of one query per (layer, sequence, query
head) over the whole cache (fp64 softmax attention on the host).

These kernels are not part of the compression step; they let a long-running
workload append, decode and compress on the GPU.  Their references are the
definitions (a row copy; softmax(scale q.K) V), written out here in numpy.
"""
import numpy as np
import pytest

import kara_inputs as ki

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _geom(rng, n_seqs, Hq, Hkv, d, dtype, bs, lens, max_blocks, extra_pages=8):
    need = [min(max_blocks, -(-int(L) // bs)) for L in lens]
    num_pages = int(sum(need)) + extra_pages
    perm = rng.permutation(num_pages)
    table = np.full((n_seqs, max_blocks), -1, dtype=np.int32)
    c = 0
    for s in range(n_seqs):
        table[s, :need[s]] = perm[c:c + need[s]]
        c += need[s]
    p = dict(window=64, buffer=0, budget=16, chunk_budget=4, max_chunk_len=4, head_dim=d, n_q_heads=Hq,
             n_kv_heads=Hkv, block_size=bs, num_pages=num_pages, max_blocks_per_seq=max_blocks, dtype=dtype,
             scale=0.0)
    return p, table, perm[c:].astype(np.int32)


def _f64(a, dtype):
    if dtype == "bf16":
        return (a.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    return a.astype(np.float64)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("f32", 4, 1, 64), ("bf16", 32, 8, 128), ("bf16", 40, 8, 128),
                                             ("bf16", 16, 1, 64), ("f32", 8, 2, 128)])
def test_decode_attention(dtype, Hq, Hkv, d):
    from paper_2607_01237_amd import kara
    _need_gpu()
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(Hq * 131 + d)
    bs, L = 16, 2
    lens = np.array([1, 255, 256, 257, 700, 0, 900, 33], dtype=np.int32)
    max_len = 800                               # the 900-token sequence is over it: zero rows
    p, table, _ = _geom(rng, len(lens), Hq, Hkv, d, dtype, bs, lens, max_blocks=64)
    print(f"\n[case] decode {dtype} Hq={Hq} Hkv={Hkv} d={d}", flush=True)
    params = kara.make_params(p, len(lens))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cpu").manual_seed(5)
    kp = [torch.randn((p["num_pages"], Hkv, bs, d), generator=g).to(dt) for _ in range(L)]
    vp = [torch.randn((p["num_pages"], Hkv, bs, d), generator=g).to(dt) for _ in range(L)]
    # seq 7 is not listed; len(lens) and -1 are indices outside the table (zero rows)
    seqs = np.array([5, 0, 3, 1, 4, 2, 6, len(lens), -1], dtype=np.int32)
    n = len(seqs)
    q = torch.randn((L, n, Hq, d), generator=g).to(dt)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    out = torch.full((L, n, Hq, d), float("nan"), dtype=torch.float32, device=dev)
    ws = torch.empty(kara.decode_workspace_size(params, n, L, max_len), dtype=torch.uint8, device=dev)
    kpd, vpd = [t.to(dev) for t in kp], [t.to(dev) for t in vp]
    kara.decode_attention(params, T(seqs), q.to(dev), kpd, vpd, T(table), T(lens), max_len, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()

    G = Hq // Hkv
    scale = 1.0 / np.sqrt(d)
    qh = _f64(ki.raw_numpy(q), dtype)
    worst = 0.0
    for l in range(L):
        kh, vh = _f64(ki.raw_numpy(kp[l]), dtype), _f64(ki.raw_numpy(vp[l]), dtype)
        for j, s in enumerate(seqs):
            if s < 0 or s >= len(lens):
                assert (got[l, j] == 0).all(), f"sequence index {s} is outside the table: zero rows"
                continue
            n_tok = int(lens[s])
            if n_tok == 0 or n_tok > max_len:
                assert (got[l, j] == 0).all(), f"seq {s} should give zero rows"
                continue
            pos = np.arange(n_tok)
            pg, sl = table[s, pos // bs], pos % bs
            for hq in range(Hq):
                K, V = kh[pg, hq // G, sl], vh[pg, hq // G, sl]
                x = scale * (K @ qh[l, j, hq])
                w = np.exp(x - x.max())
                want = (w / w.sum()) @ V
                err = np.abs(got[l, j, hq] - want)
                worst = max(worst, float(err.max()))
                assert (err <= 1e-4 + 1e-4 * np.abs(want)).all(), (l, j, hq, float(err.max()))
    print(f"[case] ok: max abs err {worst:.2e}", flush=True)


@pytest.mark.parametrize("dtype,Hq,Hkv,d,n,L,bs,max_len", [
    ("bf16", 8, 8, 64, 32, 8, 16, 1100),     # 2048 units: 1024-key splits, two of them, one query head each
    ("f32", 4, 2, 64, 32, 24, 7, 1100),      # 1536 units: 512-key splits, 16-key blocks, odd pages
    ("bf16", 6, 2, 128, 4, 1, 16, 1100),     # 8 units: 256-key splits, G = 3 of four accumulators
    ("bf16", 16, 2, 128, 4, 1, 24, 800),     # G = 8
    ("f32", 32, 2, 128, 4, 1, 16, 600),      # G = 16 in fp32: one buffer of keys
    ("bf16", 8, 8, 64, 32, 24, 16, 200),     # one split: no combine, zero rows from the split kernel
])
def test_decode_splits(dtype, Hq, Hkv, d, n, L, bs, max_len):
    # the split sizes (by units and max_len) and their edges: sequences that
    # end inside the first split, at its end and one past it, partial 16-key
    # tiles and 32-key blocks, an empty sequence, one over max_len.  Bound as
    # above: fp32 logits are off by at most d 2^-24 sum |q k| / sqrt(d), about
    # 2e-5 here, and an output by twice that times the largest value.
    from paper_2607_01237_amd import kara
    _need_gpu()
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n * 7 + d)
    edges = [1, 15, 16, 17, 31, 33, 127, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, max_len, max_len + 1, 0]
    lens = np.array([min(edges[i % len(edges)], max_len + 1) for i in range(n)], dtype=np.int32)
    if n < len(edges):
        lens[:] = [257, max_len, 33, 512][:n]
    p, table, _ = _geom(rng, n, Hq, Hkv, d, dtype, bs, lens, max_blocks=-(-(max_len + 1) // bs))
    print(f"\n[case] decode splits {dtype} {Hq}/{Hkv} d={d} n={n} L={L} max_len={max_len}", flush=True)
    params = kara.make_params(p, n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(9)
    R = lambda *shape: torch.randn(shape, generator=g, device=dev).to(dt)  # noqa: E731
    kp, vp = ([R(p["num_pages"], Hkv, bs, d) for _ in range(L)] for _ in range(2))
    q = R(L, n, Hq, d)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    out = torch.full((L, n, Hq, d), float("nan"), dtype=torch.float32, device=dev)
    ws = torch.full((kara.decode_workspace_size(params, n, L, max_len),), 255, dtype=torch.uint8, device=dev)
    kara.decode_attention(params, T(np.arange(n, dtype=np.int32)), q, kp, vp, T(table), T(lens), max_len, out, ws)
    torch.cuda.synchronize()
    tab = T(table.astype(np.int64))
    for l in (0, L - 1):
        for j in range(n):
            nt = int(lens[j])
            if nt == 0 or nt > max_len:
                assert (out[l, j] == 0).all(), f"seq {j} should give zero rows"
                continue
            pos = torch.arange(nt, device=dev)
            K, V = (t[l][tab[j][pos // bs], :, pos % bs].double().permute(1, 0, 2).contiguous() for t in (kp, vp))
            x = torch.matmul(q[l, j].double().view(Hkv, Hq // Hkv, d) / d ** 0.5, K.transpose(1, 2).contiguous())
            want = torch.matmul(torch.softmax(x, dim=2), V).view(Hq, d)
            err = (out[l, j].double() - want).abs()
            assert bool((err <= 1e-4 + 1e-4 * want.abs()).all()), (l, j, nt, float(err.max()))
    print("[case] ok", flush=True)


@pytest.mark.parametrize("dtype,Hq,Hkv,d,max_len", [
    ("bf16", 40, 8, 128, 2100),   # 4096 units: 1024-key splits of 16-key blocks, three of them
    ("f32", 32, 8, 64, 2100),
    ("bf16", 32, 2, 128, 8300),   # G = 16; 1024 units, nine 1024-key splits
])
def test_decode_full_chip(dtype, Hq, Hkv, d, max_len):
    # enough workgroups for every wave slot: the waits inside the kernel must
    # not depend on how many waves a SIMD holds.  Bound as above.
    from paper_2607_01237_amd import kara
    _need_gpu()
    dev = torch.device("cuda:0")
    n, L, bs = 128, 4, 16
    rng = np.random.default_rng(d + Hq)
    lens = rng.integers(max_len - 1100, max_len + 1, n).astype(np.int32)
    p, table, _ = _geom(rng, n, Hq, Hkv, d, dtype, bs, lens, max_blocks=-(-max_len // bs))
    print(f"\n[case] decode full chip {dtype} {Hq}/{Hkv} d={d} n={n} L={L} max_len={max_len}", flush=True)
    params = kara.make_params(p, n)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(3)
    kp, vp, q = (torch.randn(shape, generator=g, device=dev).to(dt)
                 for shape in [(p["num_pages"], Hkv, bs, d)] * 2 + [(L, n, Hq, d)])
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    out = torch.full((L, n, Hq, d), float("nan"), dtype=torch.float32, device=dev)
    ws = torch.full((kara.decode_workspace_size(params, n, L, max_len),), 255, dtype=torch.uint8, device=dev)
    kara.decode_attention(params, T(np.arange(n, dtype=np.int32)), q, [kp] * L, [vp] * L, T(table), T(lens), max_len, out, ws)
    torch.cuda.synchronize()
    tab = T(table.astype(np.int64))
    for j in range(n):
        pos = torch.arange(int(lens[j]), device=dev)
        K, V = (t[tab[j][pos // bs], :, pos % bs].double().permute(1, 0, 2).contiguous() for t in (kp, vp))
        for l in range(L):
            x = torch.matmul(q[l, j].double().view(Hkv, Hq // Hkv, d) / d ** 0.5, K.transpose(1, 2).contiguous())
            want = torch.matmul(torch.softmax(x, dim=2), V).view(Hq, d)
            err = (out[l, j].double() - want).abs()
            assert bool((err <= 1e-4 + 1e-4 * want.abs()).all()), (l, j, float(err.max()))
    print("[case] ok", flush=True)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
def test_kv_append(dtype, d):
    from paper_2607_01237_amd import kara
    _need_gpu()
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(17)
    bs, L, Hkv, n_new, max_blocks = 16, 2, 2, 37, 12
    lens = np.array([0, 15, 16, 100, 150, 40, 3, 160], dtype=np.int32)
    # map the blocks the appended tokens need, except where a case says not to
    p, table, spare = _geom(rng, len(lens), 4 * Hkv, Hkv, d, dtype, bs, lens + n_new, max_blocks)
    print(f"\n[case] append {dtype} d={d}", flush=True)
    table[5, (40 + n_new - 1) // bs] = -1          # sequence 5: last new position unmapped
    # sequence 7: 160 + 37 > 12 * 16 tokens
    seqs = np.array([3, 0, 5, 9, 1, 6, 6, 7, 2, 4], dtype=np.int32)
    want_status = np.array([0, 0, kara.SEQ_BAD_PAGE, kara.SEQ_BAD_INDEX, 0, kara.SEQ_DUP_TRIGGER,
                            kara.SEQ_DUP_TRIGGER, kara.SEQ_BAD_WINDOW, 0, 0], dtype=np.int32)
    params = kara.make_params(p, len(lens))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cpu").manual_seed(9)
    kp = [torch.randn((p["num_pages"], Hkv, bs, d), generator=g).to(dt) for _ in range(L)]
    vp = [torch.randn((p["num_pages"], Hkv, bs, d), generator=g).to(dt) for _ in range(L)]
    n = len(seqs)
    k_new = torch.randn((L, n, n_new, Hkv, d), generator=g).to(dt)
    v_new = torch.randn((L, n, n_new, Hkv, d), generator=g).to(dt)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    kpd, vpd = [t.to(dev) for t in kp], [t.to(dev) for t in vp]
    sl_d, st_d = T(lens), torch.full((n,), -7, dtype=torch.int32, device=dev)
    kara.kv_append(params, T(seqs), k_new.to(dev), v_new.to(dev), kpd, vpd, T(table), sl_d, st_d)
    torch.cuda.synchronize()
    st = st_d.cpu().numpy()
    assert np.array_equal(st, want_status), st

    want_lens = lens.copy()
    want_k = [ki.raw_numpy(t).copy() for t in kp]
    want_v = [ki.raw_numpy(t).copy() for t in vp]
    kn, vn = ki.raw_numpy(k_new), ki.raw_numpy(v_new)
    for j, s in enumerate(seqs):
        if want_status[j] != 0:
            continue
        pos = lens[s] + np.arange(n_new)
        pg, slot = table[s, pos // bs], pos % bs
        for l in range(L):
            for h in range(Hkv):
                want_k[l][pg, h, slot] = kn[l, j, :, h]
                want_v[l][pg, h, slot] = vn[l, j, :, h]
        want_lens[s] += n_new
    assert np.array_equal(sl_d.cpu().numpy(), want_lens)
    for l in range(L):
        assert np.array_equal(ki.raw_numpy(kpd[l]).view(np.uint8), want_k[l].view(np.uint8)), f"K pool {l}"
        assert np.array_equal(ki.raw_numpy(vpd[l]).view(np.uint8), want_v[l].view(np.uint8)), f"V pool {l}"
    print("[case] ok", flush=True)


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 8, 2, 128), ("bf16", 4, 2, 64), ("f32", 4, 2, 64), ("f32", 32, 2, 128)])
def test_decode_of_infinite_logits(dtype, Hq, Hkv, d):
    # keys whose logits are -inf weigh nothing, also where a wave's first block
    # or a whole split holds no others; all keys -inf, a +inf or a NaN give NaN
    # as the softmax does, in their own sequence and KV head alone.  Tolerance
    # as above (finite logits are of the same size).
    from paper_2607_01237_amd import kara
    _need_gpu()
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(d)
    bs, inf = 16, float("inf")
    # (length, [(first, last, value of the keys' element 0, in KV head 1 alone)])
    cases = [(40, [(16, 32, -inf, False)]), (40, [(0, 16, -inf, False)]), (64, [(16, 64, -inf, True)]),
             (300, [(0, 256, -inf, False)]), (1100, [(0, 1099, -inf, False)]), (700, [(32, 96, -inf, True), (256, 512, -inf, False)]),
             (90, [(0, 90, -inf, True)]), (600, [(0, 600, -inf, False)]), (500, [(300, 301, inf, True)]),
             (333, [(7, 8, float("nan"), True)]), (200, [])]
    lens = np.array([c[0] for c in cases], dtype=np.int32)
    p, table, _ = _geom(rng, len(lens), Hq, Hkv, d, dtype, bs, lens, max_blocks=80)
    print(f"\n[case] decode of infinite logits {dtype} {Hq}/{Hkv} d={d}", flush=True)
    params = kara.make_params(p, len(lens))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cpu").manual_seed(6)
    kp, vp = (torch.randn((p["num_pages"], Hkv, bs, d), generator=g).to(dt) for _ in range(2))
    n = len(lens)
    q = torch.randn((1, n, Hq, d), generator=g).to(dt)
    q[..., 0] = q[..., 0].abs() + 0.5
    for s, (_, spans) in enumerate(cases):
        for lo, hi, value, one_head in spans:
            for pos in range(lo, hi):
                kp[table[s, pos // bs], (1 if one_head else slice(None)), pos % bs, 0] = value
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    max_len = 1200
    out = torch.full((1, n, Hq, d), -3.0, dtype=torch.float32, device=dev)
    ws = torch.empty(kara.decode_workspace_size(params, n, 1, max_len), dtype=torch.uint8, device=dev)
    kara.decode_attention(params, T(np.arange(n, dtype=np.int32)), q.to(dev), [kp.to(dev)], [vp.to(dev)], T(table), T(lens),
                          max_len, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().double()[0]
    G = Hq // Hkv
    for s in range(n):
        pos = np.arange(lens[s])
        K, V = (t[table[s, pos // bs], :, pos % bs].double() for t in (kp, vp))     # [len][Hkv][d]
        for h in range(Hkv):
            x = (q[0, s, h * G:(h + 1) * G].double() @ K[:, h].T) / d ** 0.5
            want = torch.softmax(x, -1) @ V[:, h]
            one = got[s, h * G:(h + 1) * G]
            assert torch.equal(one.isnan(), want.isnan()), (s, h)
            ok = ~want.isnan()
            assert ((one - want).abs()[ok] <= 1e-4 + 1e-4 * want.abs()[ok]).all(), (s, h)


@pytest.mark.parametrize("n_new", [1, 16, 32, 33])
@pytest.mark.parametrize("dtype,Hkv,d,bs", [("bf16", 8, 128, 16), ("f32", 3, 64, 7)])
def test_kv_append_lengths(n_new, dtype, Hkv, d, bs):
    # both forms of the append (the check inside the copying and committing
    # workgroups up to 32 tokens, a kernel of its own above), every status
    # bit and its combinations; unflagged rows land bit for bit, nothing
    # else changes
    from paper_2607_01237_amd import kara
    _need_gpu()
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n_new)
    L, max_blocks = 2, -(-(100 + 40) // bs)
    cap = max_blocks * bs
    lens = np.array([0, bs - 1, bs, 60, 50, 40, 3, cap - n_new, cap - n_new + 1, 44], dtype=np.int32)
    p, table, _ = _geom(rng, len(lens), Hkv, Hkv, d, dtype, bs, np.minimum(lens + n_new, cap), max_blocks)
    table[5, (40 + n_new - 1) // bs] = p["num_pages"]        # past the pool
    table[9, 44 // bs] = -1
    seqs = np.array([3, 0, 5, 12, 1, 6, 6, 7, 2, 4, 8, 9, 9, -1], dtype=np.int32)
    dup, page, window, index = kara.SEQ_DUP_TRIGGER, kara.SEQ_BAD_PAGE, kara.SEQ_BAD_WINDOW, kara.SEQ_BAD_INDEX
    want = np.array([0, 0, page, index, 0, dup, dup, 0, 0, 0, window, dup | page, dup | page, index], dtype=np.int32)
    print(f"\n[case] append {dtype} d={d} n_new={n_new}", flush=True)
    params = kara.make_params(p, len(lens))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(3)
    R = lambda *shape: torch.randn(shape, generator=g, device=dev).to(dt)  # noqa: E731
    n = len(seqs)
    kp, vp = ([R(p["num_pages"], Hkv, bs, d) for _ in range(L)] for _ in range(2))
    k0, v0 = [t.clone() for t in kp], [t.clone() for t in vp]
    k_new, v_new = R(L, n, n_new, Hkv, d), R(L, n, n_new, Hkv, d)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    sl, st = T(lens), torch.full((n,), -7, dtype=torch.int32, device=dev)
    kara.kv_append(params, T(seqs), k_new, v_new, kp, vp, T(table), sl, st)
    torch.cuda.synchronize()
    assert np.array_equal(st.cpu().numpy(), want), st
    want_lens = lens.copy()
    for j, s in enumerate(seqs):
        if want[j]:
            continue
        pos = lens[s] + np.arange(n_new)
        pg, slot = T(table[s, pos // bs].astype(np.int64)), T((pos % bs).astype(np.int64))
        for l in range(L):
            k0[l][pg, :, slot] = k_new[l, j]
            v0[l][pg, :, slot] = v_new[l, j]
        want_lens[s] += n_new
    assert np.array_equal(sl.cpu().numpy(), want_lens)
    for l in range(L):
        assert torch.equal(kp[l], k0[l]) and torch.equal(vp[l], v0[l]), f"pools of layer {l}"
    print("[case] ok", flush=True)
