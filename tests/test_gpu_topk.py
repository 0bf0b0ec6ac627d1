"""GPU parity of step 1 (lilicorr_topk) against the oracle: ids bit-exact, logp within 1e-5.

Every row of every workload: configs 0-2 directly, configs 3-4 (full size, the benchmark's
launch configuration) against the oracle chain of every request, computed on a thread pool.
Edge cases: ragged and tiny vocabularies, K = 1 and K = 64, exact ties, signed zeros, -inf, rows
split over several workgroups, fp32 and bf16 logits. Also: forced expiry of the kernel's bounded
waits (reported, never silent), bit-identical repeated calls, and the vocabulary-sharded layout
(per-shard top-K merged on the host) against the unsharded result.
"""
import numpy as np
import pytest
import torch

import oracle
from parity import assert_close, assert_equal, to_np

pytestmark = pytest.mark.gpu


def _run(lib, logits_cpu, K):
    x = logits_cpu.cuda()
    ids, logp = lib.topk(x, K)
    torch.cuda.synchronize()
    return to_np(ids), to_np(logp)


def _check_rows(lib, logits_cpu, K, rows=None, what=""):
    gi, gl = _run(lib, logits_cpu, K)
    N, B, V = logits_cpu.shape
    x = to_np(logits_cpu).reshape(N * B, V)
    gi = gi.reshape(N * B, K)
    gl = gl.reshape(N * B, K)
    rows = range(N * B) if rows is None else rows
    for r in rows:
        ri, rl = oracle.topk(x[r][None, None], K)
        assert_equal(gi[r], ri[0, 0], f"{what} ids row {r}")
        assert_close(gl[r], rl[0, 0], f"{what} logp row {r}")


@pytest.mark.parametrize("cfg_index", [0, 1, 2])
def test_topk_configs_full(lib, cfg_inputs, cfg_index):
    cfg, inp = cfg_inputs(cfg_index)
    print(f"topk config {cfg_index} {cfg.name}", flush=True)
    gi, gl = _run(lib, inp["logits"], cfg.K)
    ri, rl = oracle.topk(to_np(inp["logits"]), cfg.K)
    assert_equal(gi, ri, f"cfg{cfg_index} ids")
    assert_close(gl, rl, f"cfg{cfg_index} logp")


@pytest.mark.parametrize("cfg_index", [3, 4])
def test_topk_full_size_all_rows(lib, cfg_inputs, oracle_chain, cfg_index):
    cfg, inp = cfg_inputs(cfg_index)
    print(f"topk config {cfg_index} {cfg.name}", flush=True)
    gi, gl = _run(lib, inp["logits"], cfg.K)
    r = oracle_chain(cfg_index)
    assert_equal(gi, r["ids"], f"cfg{cfg_index} ids ({cfg.N * cfg.B} rows)")
    assert_close(gl, r["logp"], f"cfg{cfg_index} logp")


def _bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16)


EDGE = [
    # (N, B, V, K, kind)
    (1, 1, 1, 1, "normal"),
    (1, 2, 7, 7, "normal"),
    (2, 3, 63, 5, "normal"),
    (1, 4, 1000, 64, "normal"),
    (2, 2, 32001, 16, "normal"),
    (1, 3, 32001, 1, "normal"),
    (3, 5, 70001, 33, "ties"),
    (1, 2, 5000, 8, "equal"),
    (1, 2, 3000, 20, "zeros"),
    (2, 2, 4099, 10, "neginf"),
    (1, 16, 151936, 8, "normal"),  # few rows in parts: short segments (fp32), row kernel (bf16)
    (1, 1, 262144, 64, "ties"),
    # whole rows of the row kernel with exact ties at the threshold, or few values above -inf
    (1, 2, 20000, 8, "equal"),
    (1, 2, 20000, 20, "zeros"),
    (2, 2, 20001, 10, "neginf"),
    (1, 3, 30000, 12, "maskblock"),  # whole tiles at -inf next to finite ones
    (1, 1, 20000, 64, "ties"),
    # rows in parts of 32768 and more logits + merge
    (2, 16, 151936, 16, "normal"),
    # the same at K = 64: 576 partial keys
    (1, 1, 300000, 64, "normal"),
    # one workgroup per compute unit
    (1, 256, 10000, 4, "normal"),
]


def _edge_logits(N, B, V, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "normal":
        x = rng.standard_normal((N, B, V)) * 2
    elif kind == "ties":
        x = rng.integers(-20, 21, size=(N, B, V)) * 0.25
    elif kind == "equal":
        x = np.full((N, B, V), 1.5)
    elif kind == "zeros":
        x = rng.choice([-0.0, 0.0, -1.0], size=(N, B, V))
    elif kind == "maskblock":
        x = rng.standard_normal((N, B, V))
        x[..., : V // 2] = -np.inf
        x[..., -1] = 3.0
    elif kind == "neginf":
        x = rng.standard_normal((N, B, V))
        x[rng.random((N, B, V)) < 0.9] = -np.inf
        x[..., 0] = 0.5
    return x.astype(np.float32)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("case", range(len(EDGE)))
def test_topk_edge_cases(lib, case, dtype):
    N, B, V, K, kind = EDGE[case]
    print(f"topk edge {EDGE[case]} {dtype}", flush=True)
    x = _edge_logits(N, B, V, kind, case)
    t = _bf16(x) if dtype == "bf16" else torch.from_numpy(x)
    _check_rows(lib, t, K, None, f"edge{case}-{dtype}")


def test_topk_workspace_shared_across_paths(lib):
    """One zero-filled workspace through row-kernel calls, split and whole, in turn: every call
    matches the same call on a fresh workspace bit for bit."""
    shapes = [(1, 16, 151936, 8), (2, 16, 151936, 16), (1, 256, 10000, 4), (4, 16, 151936, 16),
              (1, 16, 151936, 8), (1, 3, 30000, 12)]
    need = max(lib.lilicorr_topk_workspace_bytes(N, B, V, K) for N, B, V, K in shapes)
    ws = torch.zeros((need + 15) // 16 * 16, dtype=torch.uint8, device="cuda")
    rng = np.random.default_rng(17)
    for i, (N, B, V, K) in enumerate(shapes):
        print(f"topk shared workspace call {i}: N={N} B={B} V={V} K={K}", flush=True)
        x = _bf16(rng.standard_normal((N, B, V)) * 2).cuda()
        ids, logp = lib.topk(x, K, workspace=ws)
        ids0, logp0 = lib.topk(x, K)
        torch.cuda.synchronize()
        assert_equal(to_np(ids), to_np(ids0), f"call {i} ids")
        assert_equal(to_np(logp), to_np(logp0), f"call {i} logp")
    assert lib.topk_wait_status(ws) == 0


def test_topk_sparse_finite_row(lib):
    # fewer than K finite logits: the -inf candidates follow by id
    x = np.full((1, 2, 600), -np.inf, np.float32)
    x[0, 0, [5, 400]] = [1.0, 2.0]
    x[0, 1, 599] = -3.0
    _check_rows(lib, torch.from_numpy(x), 4, None, "sparse")


def test_topk_rejects_bad_arguments(lib):
    x = torch.zeros(1, 1, 10, device="cuda", dtype=torch.bfloat16)
    with pytest.raises(lib.LilicorrError):
        lib.topk(x, 11)
    with pytest.raises(lib.LilicorrError):
        lib.topk(x, 65)
    with pytest.raises(lib.LilicorrError):
        lib.topk(x, 0)


# ---- confidence features from the same pass (lilicorr_topk_features) ---------------------------

def _features(lib, logits_cpu, K):
    ids, logp, feat = lib.topk(logits_cpu.cuda(), K, features=True)
    torch.cuda.synchronize()
    return to_np(ids), to_np(logp), to_np(feat)


@pytest.mark.parametrize("cfg_index", [0, 1, 2, 3, 4])
def test_topk_features_configs(lib, cfg_inputs, oracle_chain, cfg_index):
    """ids / logp as lilicorr_topk gives them; features against the oracle's from its own top-K
    (config 1 splits each row over several workgroups: the merge kernel writes them)."""
    cfg, inp = cfg_inputs(cfg_index)
    print(f"features config {cfg_index} {cfg.name}", flush=True)
    gi, gl, gf = _features(lib, inp["logits"], cfg.K)
    ri, rl = lib.topk(inp["logits"].cuda(), cfg.K)
    torch.cuda.synchronize()
    assert_equal(gi, to_np(ri), "ids with and without features")
    assert_equal(gl, to_np(rl), "logp with and without features")
    if cfg.N <= 16:
        oi, ol = oracle.topk(to_np(inp["logits"]), cfg.K)
        of = oracle.candidate_features(ol)
    else:  # every request, from the session's oracle chain
        r = oracle_chain(cfg_index)
        oi, of = r["ids"], r["feat"]
    assert_equal(gi, oi, "ids")
    assert_close(gf, of, "features")


@pytest.mark.parametrize("K", [1, 3, 64])
def test_topk_features_ties_and_small_k(lib, K):
    g = torch.Generator().manual_seed(K)
    x = torch.randn(2, 5, 3000, generator=g) * 3
    x[:, :, 10:20] = x.max(-1, keepdim=True).values + 1.0  # ten-way tie at the top
    xb = x.to(torch.bfloat16)
    gi, gl, gf = _features(lib, xb, K)
    oi, ol = oracle.topk(to_np(xb), K)
    assert_equal(gi, oi, "ids")
    assert_close(gf, oracle.candidate_features(ol), "features")
    assert (gf[..., :min(K, 10), 2] == 0).all()  # tied with the top: zero gap


# ---- the row kernel: waves per workgroup, rows split over workgroups, thresholds from maxima -------

ROW_CASES = [
    # (rows, V, K, kind): short rows (streaming), then 4, 8 and 16 waves a workgroup by V, ragged ends,
    # K past the group maxima
    (3, 1, 1, "normal"), (2, 65, 64, "normal"), (5, 2049, 7, "normal"), (3, 4095, 33, "ties"),
    (3, 8193, 64, "normal"), (2, 16385, 16, "normal"), (2, 32769, 64, "normal"),
    # split over 3 (fp32: 8 streaming) and 8 workgroups, and two of them from 196608 logits
    (70, 98310, 2, "normal"), (1, 262147, 50, "ties"), (90, 196609, 3, "normal"),
    # many short rows
    (257, 2100, 9, "normal"), (641, 700, 5, "ties"), (1024, 600, 17, "normal"),
    # few long rows: short segments, row kernel in 4 parts (fp32: 10 streaming), short segments
    (3, 65537, 8, "normal"), (31, 131075, 2, "ties"), (2, 99991, 33, "normal"),
    # streaming: whole rows by V against K from 257 rows, four and two workgroups a row; beside them
    # the row kernel below 3500 K (600 rows, bf16)
    (261, 28003, 4, "normal"), (513, 14003, 4, "ties"), (600, 13999, 7, "normal"),
    (258, 200007, 2, "normal"), (513, 200003, 9, "normal"),
    (1030, 52001, 17, "normal"),
    # every tile above the last threshold, all the best logits in one lane's groups, one value,
    # fewer finite logits than K, negative thresholds
    (2, 20011, 24, "ascending"), (2, 40000, 40, "one lane"), (2, 40001, 64, "equal"),
    (2, 20000, 12, "few finite"), (2, 33001, 16, "negative"),
]


def _row_logits(rows, V, kind):
    g = np.random.default_rng(V + rows)
    x = g.standard_normal((rows, V)).astype(np.float32) * 2
    if kind == "ties":
        x = np.round(x * 2) / 2
    elif kind == "ascending":
        x = np.linspace(-4, 60, V, dtype=np.float32) + np.zeros((rows, 1), np.float32)
    elif kind == "one lane":  # lane 5 of every wave's tiles: ids 40 .. 47 of each 512 (bf16)
        x[:, (np.arange(V) // 8) % 64 == 5] += 20
    elif kind == "equal":
        x[:] = -1.5
    elif kind == "few finite":
        x[:] = -np.inf
        x[:, [7, V // 2, V - 1]] = [3.0, -2.0, 0.0]
    elif kind == "negative":
        x = -np.abs(x) - 1
    return torch.from_numpy(x[None])


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows,V,K,kind", ROW_CASES)
def test_topk_row_kernel(lib, rows, V, K, kind, bf16):
    print(f"row kernel rows={rows} V={V} K={K} {kind} bf16={bf16}", flush=True)
    x = _row_logits(rows, V, kind)
    x = x.to(torch.bfloat16) if bf16 else x
    step = max(1, rows // 24)
    _check_rows(lib, x, K, range(0, rows, step), f"{kind} V={V} K={K}")
    # the same call again gives the same bits
    a, b = _run(lib, x, K), _run(lib, x, K)
    assert_equal(a[0], b[0], "ids repeat")
    assert np.array_equal(a[1].view(np.int32), b[1].view(np.int32))


# ---- every way a row is split, the merge kernel's paths, the lines of the plan ---------------------

SPLIT_CASES = [
    # short segments: both ends of their range, ties at the threshold (lane maxima all equal: the id
    # search), more than 64 candidates, whole segments at -inf beside finite ones
    (2, 70000, 4, "normal"), (2, 98305, 33, "ties"), (1, 524288, 48, "normal"),
    (26, 155648, 4, "maskblock"), (2, 70000, 4, "equal"), (3, 8193, 41, "ties"),
    (2, 70001, 20, "few finite"), (1, 120000, 40, "zeros"),
    # row kernel in parts: a part with no finite logit, more candidates than one wave ranks, and more
    # than 2048 partial keys
    (3, 98310, 12, "maskblock"), (2, 300000, 64, "63 a part"), (1, 1200000, 64, "normal"),
    (1, 1200000, 64, "maskblock"),
    # streaming in parts: 257 to 340 rows, 513 to 640, fp32 with K = 2 (bf16: row kernel in parts)
    (258, 200007, 2, "maskblock"), (513, 200003, 9, "maskblock"), (60, 65539, 2, "maskblock"),
]

LINE_CASES = [
    # short rows: streaming up to 2560 logits (1024 above K = 56), 4608 or 8192 up to K = 4
    (3, 2560, 56, "normal"), (3, 2561, 56, "ties"), (2, 1025, 57, "normal"), (2, 8192, 4, "normal"),
    (2, 8193, 1, "normal"),
    # more than 64 and more than 128 survivors to rank
    (5, 10000, 52, "normal"), (5, 10000, 64, "ties"),
    # eight waves (257 rows), four (641, 1024); up to 512 rows either side of 7000 K (bf16) and 4000 K
    # (fp32), above of 1000 K (fp32, K = 7)
    (257, 9000, 9, "normal"), (641, 4990, 5, "ties"), (1024, 5000, 17, "normal"),
    (261, 28003, 5, "normal"), (261, 15999, 4, "normal"), (600, 6999, 7, "normal"),
    (600, 7000, 7, "normal"),
    # from 1152 (bf16) and 1280 (fp32) rows, either side of 4000 K and 2000 K; a fifth workgroup
    (1152, 67999, 17, "normal"), (1152, 68000, 17, "normal"), (1280, 33999, 17, "normal"),
    (1280, 34000, 17, "normal"), (1100, 3584, 40, "ties"), (1100, 4608, 33, "normal"),
    # 200000 logits: bf16 up to 512 rows, fp32 above
    (341, 199999, 8, "normal"), (341, 200001, 8, "normal"), (641, 200001, 8, "normal"),
]


def _split_logits(rows, V, K, kind):
    if kind == "maskblock":
        x = _row_logits(rows, V, "normal")
        x[..., : 2 * V // 3] = -np.inf
        x[..., -1] = 3.0
        return x
    if kind == "zeros":
        return torch.from_numpy(_edge_logits(1, rows, V, "zeros", K))
    x = _row_logits(rows, V, "normal" if kind == "63 a part" else kind)
    if kind == "63 a part":  # of the nine parts: no part's 64th key is above another's 63
        for p in range(9):
            x[..., p * ((V + 8) // 9):][..., :63] += 40
    return x


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows,V,K,kind", SPLIT_CASES + LINE_CASES)
def test_topk_plan_paths(lib, rows, V, K, kind, bf16):
    print(f"plan paths rows={rows} V={V} K={K} {kind} bf16={bf16}", flush=True)
    x = _split_logits(rows, V, K, kind)
    x = x.to(torch.bfloat16) if bf16 else x
    _check_rows(lib, x, K, range(0, rows, max(1, rows // 8)), f"{kind} rows={rows} V={V} K={K}")


def test_topk_workspace_shared_across_kernels(lib):
    """As test_topk_workspace_shared_across_paths, through short segments, rows in streaming parts,
    whole streaming rows, row-kernel parts and merged lists."""
    shapes = [(1, 16, 151936, 4), (258, 1, 200007, 2), (2, 600, 2000, 8), (1, 3, 98310, 12),
              (1, 1, 1200000, 64), (1, 16, 151936, 4)]
    need = max(lib.lilicorr_topk_workspace_bytes(N, B, V, K) for N, B, V, K in shapes)
    ws = torch.zeros((need + 15) // 16 * 16, dtype=torch.uint8, device="cuda")
    for i, (N, B, V, K) in enumerate(shapes):
        print(f"topk shared workspace call {i}: N={N} B={B} V={V} K={K}", flush=True)
        x = torch.randn(N, B, V, generator=torch.Generator().manual_seed(i)).to(torch.bfloat16).cuda()
        got = lib.topk(x, K, workspace=ws)
        fresh = lib.topk(x, K)
        torch.cuda.synchronize()
        for g, f in zip(got, fresh):
            assert_equal(to_np(g), to_np(f), f"call {i}")
    assert lib.topk_wait_status(ws) == 0


@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "fp32"])
@pytest.mark.parametrize("nan", ["every chunk", "whole tiles"])
@pytest.mark.parametrize("rows,V,K", [
    (2, 40000, 16), (3, 151936, 8), (3, 151936, 4),  # few rows, whole and in parts
    (260, 100000, 16), (1100, 50000, 17),  # waves of more than four tiles: maxima of every form
    (1100, 9000, 4)])                      # streaming
def test_topk_nan_logits(lib, rows, V, K, nan, bf16):
    """NaN logits are never candidates: the ids are those of the row with its NaNs at -inf, in every
    kernel and wherever the NaNs stand."""
    print(f"topk nan rows={rows} V={V} K={K} {nan} bf16={bf16}", flush=True)
    x = _row_logits(rows, V, "normal").to(torch.bfloat16 if bf16 else torch.float32)
    clean = x.clone()
    at = slice(None, None, 4) if nan == "every chunk" else slice(V // 2)
    clean[..., at] = -np.inf
    # set by bit pattern: a converted NaN may carry a sign, and positive ones sort above infinity
    x.view(torch.int16 if bf16 else torch.int32)[..., at] = 0x7FC0 if bf16 else 0x7FC00000
    gi, _ = _run(lib, x, K)
    clean = to_np(clean)[0]
    for r in range(0, rows, max(1, rows // 12)):
        ri, _ = oracle.topk(clean[r][None, None], K)
        assert_equal(gi[0, r], ri[0, 0], f"ids row {r}")


# ---- bounded waits: expiry is reported, never silent ---------------------------------------------

def test_topk_wait_expiry_is_reported(lib):
    """With the spin limit forced to 0 from the host, the streaming kernel's consumer gives up at
    once (every wave still runs to the kernel's end) and the workspace's status word reports it;
    the query clears the word, and with the default limit the same call is correct and clean."""
    N, B, V, K = 64, 16, 24576, 16  # 1024 rows, one workgroup per row: the streaming kernel
    g = torch.Generator().manual_seed(5)
    x = (torch.randn(N, B, V, generator=g) * 2).to(torch.bfloat16)
    xd = x.cuda()
    ws = lib.topk_workspace(N, B, V, K)
    assert lib.topk_wait_status(ws) == 0
    lib.lilicorr_set_wait_limit(0)
    try:
        lib.topk(xd, K, workspace=ws)
        torch.cuda.synchronize()
    finally:
        lib.lilicorr_set_wait_limit(-1)
    assert lib.topk_wait_status(ws) == -6
    assert lib.topk_wait_status(ws) == 0
    gi, gl = lib.topk(xd, K, workspace=ws)
    assert lib.topk_wait_status(ws) == 0
    ri, rl = oracle.topk(to_np(x), K)
    assert_equal(to_np(gi), ri, "ids after the forced expiry")
    assert_close(to_np(gl), rl, "logp after the forced expiry")


def test_topk_logp_is_deterministic(lib, cfg_inputs):
    """The exp sums' reference depends on each producer's own tiles only, so repeated calls give
    bit-identical log-probabilities (stress workload: planted peaks move the threshold early)."""
    cfg, inp = cfg_inputs(4)
    x = inp["logits"].cuda()
    a = [to_np(t) for t in lib.topk(x, cfg.K)]
    for _ in range(3):
        b = [to_np(t) for t in lib.topk(x, cfg.K)]
        assert_equal(b[0], a[0], "ids of repeated calls")
        assert_equal(b[1], a[1], "logp of repeated calls")


# ---- the vocabulary-sharded layout on one GPU ----------------------------------------------------

def test_topk_vocabulary_shards_merge(lib, cfg_inputs, oracle_chain):
    """What a tensor-parallel LM head over 8 GPUs would hand this path: each shard holds V/8 =
    18,992 columns of every slot. Each shard's lilicorr_topk runs on its own slice; the exchange
    the sharded design needs per slot is the shard's K (id + base, logit) keys and its
    log-sum-exp (recovered here from the shard's top key: lse_shard = x[id_0] - logp_shard[0]).
    Merged (keys by value desc, global id asc; lse = logsumexp over shards), they must equal the
    unsharded result of the oracle chain: ids bit-exact, logp within tolerance."""
    cfg, inp = cfg_inputs(3)
    x = inp["logits"]  # [64, 16, 151936] bf16
    N, B, V, K = cfg.N, cfg.B, cfg.V, cfg.K
    P = 8
    w = V // P
    assert w * P == V
    xb = to_np(x)  # bf16 bit patterns

    def values(gid):  # the logits at global ids, widened exactly
        bits = np.take_along_axis(xb, gid, axis=-1).astype(np.uint32) << 16
        return bits.view(np.float32).astype(np.float64)

    keys_v, keys_id, lses = [], [], []
    for p in range(P):
        sl = x[:, :, p * w:(p + 1) * w].contiguous()
        gi, gl = _run(lib, sl, K)
        gid = gi.astype(np.int64) + p * w
        xv = values(gid)
        keys_v.append(xv)
        keys_id.append(gid)
        lses.append(xv[..., 0] - gl[..., 0].astype(np.float64))
    kv = np.concatenate(keys_v, -1)
    ki = np.concatenate(keys_id, -1)
    order = np.lexsort((ki, -kv), axis=-1)[..., :K]
    ids = np.take_along_axis(ki, order, -1).astype(np.int32)
    lse = np.logaddexp.reduce(np.stack(lses, -1), axis=-1)
    logp = (np.take_along_axis(kv, order, -1) - lse[..., None]).astype(np.float32)
    r = oracle_chain(3)
    assert_equal(ids, r["ids"], "merged shard ids")
    assert_close(logp, r["logp"], "merged shard logp")
