"""GPU parity of the fused step (kara_compress_window) against the CPU oracle,
on every workload shape at sizes the oracle finishes in seconds, plus the
edge cases of the method (ragged compressible length, buffer, full budget,
alpha = 0, gamma = 3, unaligned windows, flagged sequences)."""
import sys

import numpy as np
import pytest

import kara_inputs as ki

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(cfg, **kw):
    import kara_check as kc
    _need_gpu()
    print(f"\n[case] {cfg['name']} {({k: cfg[k] for k in ('n_seqs', 'n_layers', 'window', 'buffer', 'budget')})}",
          flush=True)
    case = kc.setup(cfg, **kw)
    rep, gpu = kc.full_check(case)
    print(f"[case] ok {rep}", flush=True)
    return case, rep, gpu


def test_tiny_full():
    _run(ki.workload("tiny"))


def test_batch8_full():
    _, rep, _ = _run(ki.workload("batch8"))
    assert rep["units"] == 64


def test_qwen14b_shape_reduced():
    # the 64 x 40-layer batch at its real per-unit shape (W=2048, G=5), fewer units
    _run(ki.workload("qwen14b", n_seqs=2, n_layers=2, prefix=(4096, 6000)))


def test_qwen14b_buffer_ragged_tiles():
    # U=32: N=2016 is not a multiple of the 16-key tile; budget ceil(0.2*2016)=404
    _run(ki.workload("qwen14b", n_seqs=2, n_layers=1, buffer=32, budget=404, prefix=(100, 3000)))


def test_ragged_reduced():
    case, rep, gpu = _run(ki.workload("ragged", n_seqs=24, n_layers=2, prefix=(0, 1500)))
    assert len(case.geom.trig) < 24


def test_odd_geometry_and_flags():
    # N = 193 (ragged), d=64 bf16, block 7, unaligned starts, G=3; one
    # sequence triggered twice, one with a window past its end
    cfg = ki.workload("batch8", n_seqs=5, n_layers=2, n_q_heads=6, n_kv_heads=2, head_dim=64, window=200,
                      buffer=7, budget=39, chunk_budget=5, max_chunk_len=3, block_size=7, num_pages=600,
                      prefix=(0, 90), tail=(0, 20), key_mode="normal")
    g = ki.make_geometry(cfg)
    lens = g.seq_lens.copy()
    lens[4] = g.win_start[4] + 150          # window overruns the sequence
    _run(cfg, trig=[0, 1, 2, 3, 4, 2], seq_lens=lens)


@pytest.mark.parametrize("window,head_dim", [(40, 128), (150, 128), (330, 128), (150, 64), (1000, 64)])
def test_chunk_counts(window, head_dim):
    # 64-key chunks: one (N=40), odd counts whose last chunk is partial
    # (150 -> 3, 1000 -> 16 with d=64), and 330 -> 6 with a 10-key tail;
    # G*W not a multiple of the 512 rows of a workgroup
    budget = max(2, (window + 4) // 5)
    cfg = ki.workload("batch8", n_seqs=2, n_layers=1, window=window, budget=budget, chunk_budget=min(4, budget - 1),
                      max_chunk_len=4, head_dim=head_dim, prefix=(0, 70), tail=(0, 12), num_pages=256)
    _run(cfg)


def test_fp32_head128_mha():
    cfg = ki.workload("tiny", n_seqs=3, n_q_heads=2, n_kv_heads=2, head_dim=128, window=96, budget=20,
                      chunk_budget=6, max_chunk_len=5, num_pages=64, prefix=(3, 40), tail=(0, 9))
    _run(cfg)


@pytest.mark.parametrize("head_dim,window", [(64, 1024), (128, 512)])
def test_fp32_at_its_largest_window(head_dim, window):
    # fp32 windows hold at most 64K head-dim elements of keys: 1024 keys at
    # d = 64, 512 at d = 128 (two query heads per KV head)
    cfg = ki.workload("tiny", n_seqs=2, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, window=window,
                      budget=window // 5, chunk_budget=8, max_chunk_len=6, num_pages=256, prefix=(3, 90), tail=(0, 9))
    _run(cfg)


def test_more_layers_than_one_launch_takes():
    # 66 layers: scoring and compaction each run as two launches (64 + 2
    # layers' pool pointers), the scores and kept rows laid out across both
    cfg = ki.workload("batch8", n_seqs=2, n_layers=66, n_q_heads=2, n_kv_heads=1, window=128, budget=26,
                      chunk_budget=4, max_chunk_len=4, prefix=(0, 40), tail=(0, 7), num_pages=64)
    _run(cfg)


@pytest.mark.parametrize("budget,alpha,gamma", [(1024, 16, 8), (205, 0, 8), (300, 64, 3), (1, 0, 3)])
def test_selection_extremes(budget, alpha, gamma):
    cfg = ki.workload("batch8", n_seqs=2, budget=budget, chunk_budget=alpha, max_chunk_len=gamma)
    _run(cfg)


def test_deterministic():
    import kara_check as kc
    _need_gpu()
    cfg = ki.workload("batch8", n_seqs=3)
    a = kc.run_compress(kc.setup(cfg))
    b = kc.run_compress(kc.setup(cfg))
    for k in ("scores", "discrete", "kept", "bt", "seq_lens", "freed", "n_freed", "status"):
        assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), k


def test_bf16_long_window():
    # N = 2500: 40 64-key chunks with a 4-key tail; G=2, one KV head
    cfg = ki.workload("batch8", n_seqs=2, n_layers=1, n_q_heads=2, n_kv_heads=1, window=2500, budget=500,
                      prefix=(0, 100), tail=(0, 5), num_pages=512, key_mode="normal")
    _run(cfg)


@pytest.mark.parametrize("window,buffer", [(4096, 0), (4128, 32)])
def test_maximum_compressible_window(window, buffer):
    # N = 4096, the largest compressible length the library takes: 64 chunks
    # of 64 keys in each scoring sweep, the 16-position selection instance
    # at its limit; with a buffer, the buffer queries score as well
    cfg = ki.workload("batch8", n_seqs=2, n_layers=1, n_q_heads=2, n_kv_heads=1, window=window, buffer=buffer,
                      budget=820, prefix=(0, 100), tail=(0, 5), num_pages=1024, key_mode="normal")
    _run(cfg)



@pytest.mark.parametrize("window", [600, 1000, 1024, 1100, 1300, 1536, 1700, 1792, 2016, 2048])
def test_single_sweep_instances(window):
    # bf16, d = 128: every instance of the single-sweep scoring kernel, by
    # key tiles per wave and whether it watches for the last key: N = 600 (12),
    # 1000 (16), 1024 (16, whole), 1100 (20), 1300 (24), 1536 (24, whole), 1700
    # (28, ragged) and 1792 (28, all tiles full in the instance that watches),
    # 2016 (32), 2048 (32, whole)
    cfg = ki.workload("batch8", n_seqs=2, n_layers=1, n_q_heads=4, n_kv_heads=1, window=window,
                      budget=window // 5, prefix=(0, 100), tail=(0, 9), num_pages=600, key_mode="normal")
    _run(cfg)


@pytest.mark.parametrize("pos,scale", [(700, 16.0), (300, 16.0), (40, 16.0), (700, -16.0)])
def test_outlier_keys(pos, scale):
    # One window key per (sequence, head) scaled by 16 (exact in bf16).
    # Positive: its logits lie far above the maximum of the row's first keys,
    # where the scoring kernel takes its reference, and it takes nearly all
    # the probability of the rows it agrees with.  Its fp16 weights overflow
    # in roughly a third of the rows of every row tile, so the row sums' selector
    # products meet infinities (0 * inf: whole row tiles of NaN sums) and the
    # overflow redo has to take NaN as overflow.  Negative: its probabilities
    # sit tens of binades below the row maxima.
    import kara_check as kc
    _need_gpu()
    cfg = ki.workload("batch8", n_seqs=2, n_layers=1, key_mode="normal")
    print(f"\n[case] outlier key at window position {pos}, scale {scale}", flush=True)
    case = kc.setup(cfg)
    bs = case.p["block_size"]
    for t, s_ in enumerate(case.geom.trig):
        j = int(case.geom.win_start[s_]) + pos
        page = int(case.geom.block_table[s_, j // bs])
        case.kp[0][page, :, j % bs, :] *= scale
    case.host = kc.snapshot(case)
    rep, gpu = kc.full_check(case)
    print(f"[case] ok {rep}", flush=True)
    if scale > 0:
        # the outlier takes nearly all the probability of the rows whose dot
        # product with it is positive, about half of the G*W rows
        w = gpu["scores"][0, :, :, pos]
        assert (w > 0.25 * case.p["n_q_heads"] // case.p["n_kv_heads"] * case.p["window"]).all()


@pytest.mark.parametrize("dtype,d,window,buffer,queries", [
    ("bf16", 64, 64, 0, 0), ("bf16", 64, 65, 0, 0), ("bf16", 64, 192, 0, 0),       # 4, 8 and 12 tiles, one key part
    ("bf16", 64, 256, 1, 0), ("bf16", 64, 270, 13, 0),                             # its largest, and the first of two parts
    ("bf16", 64, 449, 0, 0), ("bf16", 64, 513, 0, 0), ("bf16", 64, 700, 31, 0),    # 16 x 2, 10 x 4 and 12 x 4 tiles
    ("bf16", 64, 897, 0, 0), ("bf16", 64, 1152, 0, 0), ("bf16", 64, 1153, 0, 0),   # 16 x 4, 18 x 4, and two sweeps past it
    ("bf16", 128, 1, 0, 0), ("bf16", 128, 512, 0, 17), ("bf16", 128, 513, 0, 0),   # one key; 512 resident, 513 streamed
    ("f32", 64, 512, 0, 0), ("f32", 64, 513, 0, 0), ("f32", 128, 256, 0, 0), ("f32", 128, 257, 0, 0),
])
@pytest.mark.parametrize("outlier", [False, True])
def test_resident_keys(dtype, d, window, buffer, queries, outlier):
    # The kernel that keeps a unit's keys in LDS, at the edges of its
    # instances (key tiles per wave x key parts) and of its range.  With an
    # outlier, the last key x 256 (exact): its logits pass the first tiles'
    # maxima by far more than 128 log2 units in a third of the rows, so
    # their sums overflow and the rows run again from the exact maximum.
    import kara_check as kc
    n = window - buffer
    budget = max(1, n // 5)
    cfg = ki.workload("batch8", n_seqs=2, n_layers=1, n_q_heads=6, n_kv_heads=2, dtype=dtype, head_dim=d, window=window,
                      buffer=buffer, budget=budget, chunk_budget=min(4, budget - 1), max_chunk_len=4, prefix=(0, 90),
                      tail=(0, 9), num_pages=256, key_mode="normal", score_queries=queries)
    _need_gpu()
    print(f"\n[case] resident keys {dtype} d={d} N={n} outlier={outlier}", flush=True)
    case = kc.setup(cfg)
    if outlier:
        bs = case.p["block_size"]
        for s_ in case.geom.trig:
            j = int(case.geom.win_start[s_]) + n - 1
            case.kp[0][int(case.geom.block_table[s_, j // bs]), :, j % bs, :] *= 256.0
        case.host = kc.snapshot(case)
    rep, _ = kc.full_check(case)
    print(f"[case] ok {rep}", flush=True)


def test_buffer_only_scoring():
    # the ablation without bidirectional attention: only the 64 buffer
    # queries score the 960 compressible keys (q holds those 64 positions)
    _run(ki.workload("buffer_only", n_seqs=3, n_layers=2, window=1024, budget=192, prefix=(0, 300)))


def test_threshold_topk_baseline():
    # Eq. (2)-(3): the whole cache (1280 tokens at the threshold) is the
    # window, its last 32 tokens score and are kept, plain top-k of 993
    case, rep, gpu = _run(ki.workload("threshold_topk", n_seqs=3, n_layers=2))
    assert (gpu["seq_lens"][case.geom.trig] == 1025).all()


def test_kvllm_serving_geometry():
    # the serving runs' geometry (App. B.1): 256-token blocks, a window of
    # three blocks with a 32-token buffer, 225 kept + 32 buffer = 257 retained
    _run(ki.workload("batch8", n_seqs=3, n_layers=2, block_size=256, window=768, buffer=32, budget=225,
                     prefix=(0, 600), tail=(0, 255), num_pages=40))


def test_wide_block_table():
    # a block-table row wider than compaction stages in LDS (8,192 words with
    # the kept rows): the instance that reads the kept indices and the table
    # from global memory for every tile
    _, rep, _ = _run(ki.workload("batch8", n_seqs=2, n_layers=2, max_blocks=8400))


@pytest.mark.parametrize("dtype,d,window,part", [
    ("bf16", 64, 240, 0), ("f32", 128, 100, 0),                                    # one key part
    ("bf16", 64, 449, 256), ("bf16", 128, 512, 256), ("f32", 128, 256, 128),       # two, of `part` keys
    ("bf16", 64, 520, 160), ("bf16", 64, 1152, 288),                               # four
    ("bf16", 64, 1200, 600), ("f32", 64, 600, 300),                                # past the kernel's range: two sweeps
])
def test_resident_keys_far_above_their_reference(dtype, d, window, part):
    # Every query finds one late key far above the first tile, where a wave
    # takes its reference: up to where its weight nearly overflows fp32 and the
    # row's 1 / sum lies below the normal range, and past it.  With several
    # key parts, also beside a part whose reference is as far above the first
    # part's, so that the two references differ by more than 2^126 while the
    # late key still holds an eighth of the row.
    import kara_check as kc
    from paper_2607_01237_amd import kara
    _need_gpu()
    print(f"\n[case] late key far above the reference, {dtype} d={d} N={window}", flush=True)
    c = kc.setup(ki.workload("batch8", n_seqs=1, n_layers=1, n_q_heads=2, n_kv_heads=1, dtype=dtype, head_dim=d,
                             window=window, budget=window // 5, chunk_budget=4, max_chunk_len=4, prefix=(5, 5), tail=(3, 3),
                             num_pages=96, key_mode="normal"))
    bs, s = c.p["block_size"], int(c.geom.trig[0])
    rows = [(int(c.geom.block_table[s, j // bs]), j % bs)
            for j in range(int(c.geom.win_start[s]), int(c.geom.win_start[s]) + window)]
    # logits = a key's first element (+ about 0.05): 8 * scale * sqrt(d / 64)
    c.q *= 0.25
    c.q[..., 0] = 8.0 * (d / 64) ** 0.5
    c.kp[0] *= 0.25
    for pg, o in rows:
        c.kp[0][pg, :, o, 0] = 0.0
    ws = torch.empty(kara.workspace_size(c.params, 1, 1), dtype=torch.uint8, device="cuda")
    late = (part if part else window) - 3
    for high in (40.0, 42.0, 60.0, 75.0, 87.0, 87.5, 88.0, 88.5, 89.0, 100.0):
        for beside in (None,) if not part else (None, high + 2.0):
            pg, o = rows[late]
            c.kp[0][pg, :, o, 0] = high
            if part:
                pg, o = rows[part + 2]
                c.kp[0][pg, :, o, 0] = beside if beside is not None else 0.0
            c.host = kc.snapshot(c)
            scores = torch.full((1, 1, 1, window), float("nan"), device="cuda")
            st = torch.full((1,), -1, dtype=torch.int32, device="cuda")
            kara.score_window(c.params, c.trig, c.q, c.kp, c.bt, c.seq_lens, c.win_start, scores, st, ws)
            torch.cuda.synchronize()
            ora, _ = kc.oracle_scores(c)
            rep = kc.check_p1(scores.cpu().numpy(), ora)
            print(f"[case] key at {high}, beside {beside}: {rep}", flush=True)
            # (2 x window rows, all but a few of their weight on the placed keys)
            assert ora[0, 0, 0, late] > 0.1 * 2 * window


@pytest.mark.parametrize("dtype,d,window", [
    ("bf16", 64, 200), ("bf16", 64, 449), ("bf16", 64, 1152), ("bf16", 128, 512), ("f32", 64, 500), ("f32", 128, 256),   # resident
    ("bf16", 128, 600), ("bf16", 128, 1100), ("bf16", 128, 1700), ("bf16", 128, 2048),                                  # single sweep
    ("bf16", 64, 1200), ("f32", 64, 600),                                                                                # two sweeps
])
def test_scores_of_infinite_and_nan_keys(dtype, d, window):
    # keys whose logits are -inf weigh nothing, also where they fill the tiles
    # a reference is taken from or all keys but one; a +inf or a NaN key, or no
    # finite one, makes its own (sequence, KV head) NaN as the softmax does, and
    # no other
    import kara_check as kc
    from paper_2607_01237_amd import kara
    _need_gpu()
    inf = float("inf")
    print(f"\n[case] infinite and NaN keys, {dtype} d={d} N={window}", flush=True)
    # per sequence and KV head: (positions, value of the keys' element 0)
    plan = [(slice(3, 4), -inf), (slice(0, 16), -inf), (slice(0, window, 2), -inf), (slice(0, window - 1), -inf),
            (slice(0, window), -inf), (slice(window // 2, window // 2 + 1), inf), (slice(window - 2, window - 1), float("nan")),
            (slice(16, 20), -inf)]
    c = kc.setup(ki.workload("batch8", n_seqs=4, n_layers=1, n_q_heads=4, n_kv_heads=2, dtype=dtype, head_dim=d,
                             window=window, budget=window // 5, chunk_budget=4, max_chunk_len=4, prefix=(5, 90), tail=(3, 9),
                             num_pages=-(-(window + 110) // 16) * 4 + 4, key_mode="normal"))
    bs = c.p["block_size"]
    c.q[..., 0] = c.q[..., 0].abs() + 0.5
    keys = torch.empty((4, 2, window, d), dtype=torch.float64)
    for s in range(4):
        pos = int(c.geom.win_start[s]) + np.arange(window)
        pg = torch.as_tensor(c.geom.block_table[s, pos // bs].astype(np.int64), device="cuda")
        sl = torch.as_tensor((pos % bs).astype(np.int64), device="cuda")
        for h in range(2):
            rows, value = plan[2 * s + h]
            c.kp[0][pg[rows], h, sl[rows], 0] = value
            keys[s, h] = c.kp[0][pg, h, sl].cpu().double()
    assert list(c.geom.trig) == [0, 1, 2, 3]
    ws = torch.empty(kara.workspace_size(c.params, 4, 1), dtype=torch.uint8, device="cuda")
    scores = torch.full((1, 4, 2, window), -1.0, device="cuda")
    st = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    kara.score_window(c.params, c.trig, c.q, c.kp, c.bt, c.seq_lens, c.win_start, scores, st, ws)
    torch.cuda.synchronize()
    assert (st == 0).all()
    got = scores.cpu().numpy()[0]
    for s in range(4):
        for h in range(2):
            x = c.q[0, s, :, 2 * h:2 * h + 2].cpu().double().reshape(-1, d) @ keys[s, h].T / d ** 0.5
            want = torch.softmax(x, -1).sum(0).numpy()
            if 2 * s + h in (4, 5, 6):
                assert np.isnan(want).all() and np.isnan(got[s, h]).all(), (s, h)
                continue
            assert np.isfinite(got[s, h]).all(), (s, h)
            assert (np.abs(got[s, h] - want) <= kc.tol(want)).all(), (s, h, float(np.abs(got[s, h] - want).max()))
