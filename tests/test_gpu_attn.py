"""GPU parity of sr_tree_verify_attn against the float64 oracle (App. B.1 Eq. (nodep))."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2608_04962_amd as sr
import synth
from helpers import dev_tensor, f64, row_rel_err, tol_for

pytestmark = pytest.mark.gpu


def _run_gpu(inp):
    t = {k: dev_tensor(inp[k]) for k in ("q", "k_cache", "v_cache", "k_tree", "v_tree")}
    out, lse = sr.tree_verify_attn(t["q"], t["k_cache"], t["v_cache"], dev_tensor(inp["block_table"]),
                                   dev_tensor(inp["ctx_len"]), t["k_tree"], t["v_tree"], dev_tensor(inp["parents"]),
                                   scale=inp["scale"])
    torch.cuda.synchronize()
    return out.cpu().numpy(), lse.cpu().numpy()


def _oracle(inp, nodes=None):
    dt = inp["dtype"]
    return oracle.tree_attention(f64(inp["q"], dt), f64(inp["k_cache"], dt), f64(inp["v_cache"], dt),
                                 inp["block_table"], inp["ctx_len"], f64(inp["k_tree"], dt), f64(inp["v_tree"], dt),
                                 inp["parents"], inp["scale"], 16, nodes=nodes)


def _check(inp, nodes=None):
    print(f"[attn] {inp['cfg'].name} B={inp['cfg'].B} T={inp['cfg'].T}", flush=True)
    out, lse = _run_gpu(inp)
    ro, rl = _oracle(inp, nodes)
    tol = tol_for(inp["dtype"])
    sel = ~np.isnan(ro[..., 0])
    assert sel.any()
    err = row_rel_err(out[sel], ro[sel])
    assert err.max() <= tol, f"max row error {err.max():.3e} > {tol}"
    # lse (natural log of the softmax normaliser): absolute error within the same bar
    lerr = np.abs(lse[sel] - rl[sel]).max()
    print(f"[parity] attention {inp['cfg'].name}: {int(sel.sum() // inp['cfg'].Hq)} nodes, max row rel err "
          f"{err.max():.2e}, max lse abs err {lerr:.2e} (bar {tol})", flush=True)
    assert lerr <= tol, f"lse error {lerr:.3e} > {tol}"
    assert np.isfinite(out).all()
    return err.max()


def test_config0_all_nodes():
    _check(synth.attn_inputs(synth.TINY_FP32, seed=0))


@pytest.mark.parametrize("seed", [0, 1])
def test_bf16_multi_chunk_ragged(seed):
    # 10 (trajectory, KV head) pairs take 32-page (512-token) chunks: contexts up to 5000 tokens run the
    # split/combine path over up to ten chunks with ragged tails
    cfg = synth.scaled(synth.SHAPE_7B, B=5, T=12, depth=4, Hq=8, Hkv=2, ctx=("uniform", 1, 5000))
    inp = synth.attn_inputs(cfg, seed=seed)
    _check(inp)


def test_bf16_long_chunks_all_nodes():
    # 512 (trajectory, KV head) pairs select 256-page prefix chunks: contexts of 2900-9000 tokens take one
    # to three chunks, with ragged tails; every node of every trajectory is compared
    cfg = synth.scaled(synth.SHAPE_7B, B=128, T=2, depth=1, ctx=("uniform", 2900, 9000))
    _check(synth.attn_inputs(cfg, seed=5))


def test_bf16_rows_over_one_block_gqa7():
    # T*G = 40*7 = 280 > 256 query rows: two row groups
    cfg = synth.scaled(synth.SHAPE_7B, B=2, T=40, depth=5, ctx=("uniform", 100, 3000))
    _check(synth.attn_inputs(cfg, seed=3))


def test_fp32_d128_and_bf16_d64():
    _check(synth.attn_inputs(synth.scaled(synth.TINY_FP32, D=128, Hq=6, Hkv=3), seed=4))
    _check(synth.attn_inputs(synth.scaled(synth.SHAPE_1P5B, dtype="bf16", B=3, D=64, ctx=("uniform", 20, 300)),
                             seed=5))


def test_one_query_head_per_kv_head():
    # G = 1 (no grouping): one 32-row block per T nodes, split prefixes with ragged tails, bf16 and fp32
    _check(synth.attn_inputs(synth.scaled(synth.SHAPE_7B, B=6, T=32, Hq=4, Hkv=4, ctx=("uniform", 900, 5000)),
                             seed=11))
    _check(synth.attn_inputs(synth.scaled(synth.SHAPE_7B, dtype="f32", B=3, T=16, Hq=2, Hkv=2,
                                          ctx=("uniform", 100, 3000)), seed=12))


def test_empty_prefix_and_single_node_tree():
    _check(synth.attn_inputs(synth.scaled(synth.TINY_FP32, ctx=("explicit", (0, 17))), seed=6))
    _check(synth.attn_inputs(synth.scaled(synth.TINY_FP32, T=1, parents=(-1,), ctx=("explicit", (0, 2049))),
                             seed=7))
    _check(synth.attn_inputs(synth.scaled(synth.SHAPE_7B, B=2, T=128, depth=6, Hq=4, Hkv=4,
                                          ctx=("uniform", 0, 40)), seed=8))


def test_invalid_inputs_give_nan_rows_only_for_that_trajectory():
    cfg = synth.scaled(synth.SHAPE_7B, B=3, T=8, depth=3, Hq=8, Hkv=2, ctx=("uniform", 40, 3000))
    inp = synth.attn_inputs(cfg, seed=9)
    inp["block_table"] = inp["block_table"].copy()
    inp["block_table"][1, 0] = inp["num_blocks"] + 5      # page id out of range
    inp["ctx_len"] = inp["ctx_len"].copy()
    inp["ctx_len"][2] = cfg.max_blocks * 16 + 1           # longer than the table
    out, lse = _run_gpu(inp)
    assert np.isnan(out[1]).all() and np.isnan(out[2]).all()
    assert np.isnan(lse[1]).all() and np.isnan(lse[2]).all()
    assert np.isfinite(out[0]).all()
    inp2 = synth.attn_inputs(cfg, seed=9)
    inp2["parents"] = inp2["parents"].copy()
    inp2["parents"][0, 3] = 5                             # not an earlier node
    out2, _ = _run_gpu(inp2)
    assert np.isnan(out2[0]).all() and np.isfinite(out2[1:]).all()
    inp3 = synth.attn_inputs(cfg, seed=9)
    inp3["ctx_len"] = inp3["ctx_len"].copy()
    inp3["ctx_len"][1] = -1                               # negative length
    out3, lse3 = _run_gpu(inp3)
    assert np.isnan(out3[1]).all() and np.isnan(lse3[1]).all()
    assert np.isfinite(out3[0]).all() and np.isfinite(out3[2]).all()


def test_deterministic():
    cfg = synth.scaled(synth.SHAPE_7B, B=4, T=16, depth=4, ctx=("uniform", 1000, 4500))
    inp = synth.attn_inputs(cfg, seed=10)
    a, la = _run_gpu(inp)
    b, lb = _run_gpu(inp)
    np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(la, lb)


def _sample_nodes(cfg, k, seed):
    rng = np.random.default_rng(seed)
    bs = rng.choice(cfg.B, size=min(k, cfg.B), replace=False)
    return [(int(b), int(u)) for b in bs for u in rng.choice(cfg.T, size=min(4, cfg.T), replace=False)]


@pytest.mark.parametrize("name,rseed", [("1.5B-shape", 1), ("7B-shape", 2), ("14B-shape-tail", 3)])
def test_full_size_sampled(name, rseed):
    cfg = synth.WORKLOADS[name]
    inp = synth.attn_inputs(cfg, seed=0)
    _check(inp, nodes=_sample_nodes(cfg, 6, rseed))


@pytest.mark.parametrize("point", synth.SWEEP_POINTS, ids=lambda p: f"B{p[0]}-T{p[1]}")
def test_sweep_points_sampled(point):
    cfg = synth.sweep_config(*point)
    inp = synth.attn_inputs(cfg, seed=0)
    _check(inp, nodes=_sample_nodes(cfg, 4, point[0]))


@pytest.mark.parametrize("T,Hq,Hkv", [(32, 32, 4), (29, 32, 4), (64, 16, 4)])
def test_bf16_rows_224_to_256(T, Hq, Hkv):
    # T*G of 256, 232 and 256 query rows per KV head: more than 224, so the rows split into two groups
    # (each keeps a wave free of query rows for the K/V transfers); contexts take one to several chunks
    cfg = synth.scaled(synth.SHAPE_7B, B=3, T=T, depth=5, Hq=Hq, Hkv=Hkv, ctx=("uniform", 100, 3000))
    _check(synth.attn_inputs(cfg, seed=11))


def _scale_values(inp, traj, fn):
    """Apply fn to the float values of trajectory traj's prefix V pages and tree V rows (bf16 bits kept)."""
    inp = dict(inp)
    vc = synth.to_f64(inp["v_cache"], "bf16")
    vt = synth.to_f64(inp["v_tree"], "bf16")
    L = int(inp["ctx_len"][traj])
    pages = inp["block_table"][traj, :-(-L // 16)]
    vc[pages] = fn(vc[pages])
    vt[traj] = fn(vt[traj])
    inp["v_cache"] = synth.as_dtype(vc.astype(np.float32), "bf16")
    inp["v_tree"] = synth.as_dtype(vt.astype(np.float32), "bf16")
    return inp


def test_bf16_v_outside_fp16_range():
    """bf16 V beyond what the fp16 product keeps: magnitudes around 1e5 (fp16 overflows past 65504), V scaled to
    around 1e-6 and 1e-30 (below fp16's normal range, so its subnormal step would dominate) and a mix of huge
    and tiny values in one trajectory. Those items are recomputed with fp32 V; the others (N(0,1) values, a
    few of them below 2^-14) keep the fp16 product; every trajectory matches the oracle."""
    cfg = synth.scaled(synth.SHAPE_7B, B=6, T=12, depth=4, Hq=8, Hkv=2, ctx=("uniform", 300, 2600))
    inp = synth.attn_inputs(cfg, seed=12)
    inp = _scale_values(inp, 1, lambda v: v * 1.0e5)
    inp = _scale_values(inp, 2, lambda v: v * 1.0e-6)
    inp = _scale_values(inp, 3, lambda v: np.where(np.arange(v.shape[-1]) % 2 == 0, v * 1.0e5, v * 1.0e-6))
    inp = _scale_values(inp, 4, lambda v: v * 1.0e-30)
    out, _ = _run_gpu(inp)
    assert np.isfinite(out).all()
    _check(inp)


def _scale_keys(inp, traj, fn):
    """Multiply trajectory traj's prefix K row of key position k by fn(k), and its tree K rows by fn(L + node)
    (bf16 bits kept)."""
    inp = dict(inp)
    kc = synth.to_f64(inp["k_cache"], "bf16")
    kt = synth.to_f64(inp["k_tree"], "bf16")
    L = int(inp["ctx_len"][traj])
    for k in range(L):
        kc[inp["block_table"][traj, k // 16], :, k % 16, :] *= fn(k)
    for u in range(kt.shape[1]):
        kt[traj, u] *= fn(L + u)
    inp["k_cache"] = synth.as_dtype(kc.astype(np.float32), "bf16")
    inp["k_tree"] = synth.as_dtype(kt.astype(np.float32), "bf16")
    return inp


def test_bf16_scores_growing_falling_and_spiking():
    """The running reference max under scores that move across tiles: keys scaled up along the context
    (every later tile's scores above the first's), scaled down along it, one key at 12x in the middle of a
    long context, and tree keys at 6x (the last tile holds the largest scores)."""
    cfg = synth.scaled(synth.SHAPE_7B, B=5, T=12, depth=4, Hq=8, Hkv=2, ctx=("uniform", 1500, 3000))
    inp = synth.attn_inputs(cfg, seed=21)
    L = inp["ctx_len"]
    inp = _scale_keys(inp, 0, lambda k: 0.05 + 5.0 * k / L[0])
    inp = _scale_keys(inp, 1, lambda k: 5.05 - 5.0 * k / L[1])
    inp = _scale_keys(inp, 2, lambda k: 12.0 if k == L[2] // 2 else 1.0)
    inp = _scale_keys(inp, 3, lambda k: 6.0 if k >= L[3] else 1.0)
    out, _ = _run_gpu(inp)
    assert np.isfinite(out).all()
    _check(inp)


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("T,Hq,Hkv,D,lens", [
    (1, 2, 2, 64, (0, 1, 63, 64, 65)),                     # one tree key; units of one to three tiles, not cut
    (65, 4, 2, 128, (0, 64, 200, 2049, 513)),              # two tree tiles; ranges that start in either
    (128, 2, 1, 64, (1000, 0, 1, 4096)),                   # the largest tree
    (8, 10, 1, 128, (3000,)),                              # one unit cut into ranges of the least length
])
def test_cut_edges(dt, T, Hq, Hkv, D, lens):
    """Ranges of 64-key tiles across units: prefixes of no, one and several tiles, ragged by one key, with trees of
    one and two tiles, and one unit over many ranges."""
    cfg = synth.scaled(synth.SHAPE_7B, dtype=dt, B=len(lens), T=T, depth=5, Hq=Hq, Hkv=Hkv, D=D, ctx=("explicit", lens))
    _check(synth.attn_inputs(cfg, seed=31))


@pytest.mark.parametrize("T,Hq,Hkv,D,lens", [
    (16, 4, 2, 128, (0, 1, 31, 32, 33, 700)),              # 32 rows, half tiles with and without a key in range
    (33, 2, 2, 128, (0, 95, 700)),                         # one row more: the kernel of whole tiles
    (4, 16, 2, 64, (5000,)),                               # two units over many ranges, merged afterwards
    (31, 2, 2, 64, (64, 0, 8 * 32 + 1, 2049)),             # 31 rows; one half tile more than a round of the waves
])
def test_f32_few_rows(T, Hq, Hkv, D, lens):
    """fp32 with at most 32 query rows per KV head: half tiles over the waves, and the first size past it."""
    cfg = synth.scaled(synth.SHAPE_7B, dtype="f32", B=len(lens), T=T, depth=3, Hq=Hq, Hkv=Hkv, D=D, ctx=("explicit", lens))
    _check(synth.attn_inputs(cfg, seed=34))


def test_many_short_units_and_wide_values():
    """More trajectories than a block has threads and many units a range, some with V outside fp16's range (those
    segments alone are recomputed)."""
    rng = np.random.default_rng(5)
    lens = tuple(int(x) for x in rng.integers(0, 330, size=600))
    cfg = synth.scaled(synth.SHAPE_7B, B=600, T=5, depth=2, Hq=4, Hkv=2, ctx=("explicit", lens))
    inp = synth.attn_inputs(cfg, seed=32)
    for b in (0, 7, 300, 599):
        inp = _scale_values(inp, b, lambda v: v * 1.0e5)
    inp = _scale_values(inp, 301, lambda v: v * 1.0e-6)
    _check(inp, nodes=[(b, u) for b in (0, 1, 7, 8, 299, 300, 301, 302, 511, 512, 598, 599) for u in range(5)])


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_least_workspace(dt):
    """A workspace of one partial result per 32-page chunk (and, for bf16, two lists of the chunks) is taken too, with
    fewer ranges; none at all for prefixes of one chunk, whose units are then not cut."""
    import ctypes as C
    from paper_2608_04962_amd import _lib
    for max_len, nch in ((1000, 2), (500, 1)):
        cfg = synth.scaled(synth.SHAPE_1P5B, dtype=dt, B=6, ctx=("uniform", max_len // 2, max_len))
        inp = synth.attn_inputs(cfg, seed=33)
        up = lambda x: -(-x // 256) * 256
        rows = 12 * nch * 96
        size = (up(rows * 512) + up(rows * 8) if nch > 1 else 0) + (up((3 + 2 * 12 * nch) * 4) if dt == "bf16" else 0)
        t = {k: dev_tensor(inp[k]) for k in ("q", "k_cache", "v_cache", "k_tree", "v_tree", "block_table", "ctx_len", "parents")}
        desc = sr.attn_desc(t["q"], t["k_cache"], t["block_table"], inp["scale"])
        assert size < _lib.lib().sr_tree_verify_attn_workspace(C.byref(desc))
        ws = torch.full((max(size, 1),), 0xAB, dtype=torch.uint8, device="cuda")
        out = torch.empty(tuple(t["q"].shape), device="cuda")
        lse = torch.empty(tuple(t["q"].shape[:3]), device="cuda")
        p = lambda x: C.c_void_p(x.data_ptr())
        st = _lib.lib().sr_tree_verify_attn(C.byref(desc), p(t["q"]), p(t["k_cache"]), p(t["v_cache"]), p(t["block_table"]),
                                            p(t["ctx_len"]), p(t["k_tree"]), p(t["v_tree"]), p(t["parents"]), p(out), p(lse),
                                            p(ws) if size else None, size, None)
        torch.cuda.synchronize()
        assert st == _lib.SR_OK, _lib.last_error()
        ro, rl = _oracle(inp)
        assert row_rel_err(out.cpu().numpy(), ro).max() <= tol_for(dt)
        assert np.abs(lse.cpu().numpy() - rl).max() <= tol_for(dt)


def _pooled_inputs(dt, B, T, Hq, Hkv, D, lens, max_blocks, pool, seed):
    """Inputs whose block tables draw their pages from a small pool, so that contexts may be as long as a table
    holds; past a trajectory's last page the table holds ids out of range."""
    rng = np.random.default_rng(seed)
    mk = lambda *s: synth.as_dtype(rng.standard_normal(s).astype(np.float32), dt)
    bt = np.full((B, max_blocks), -7, np.int32)
    for b, n in enumerate(lens):
        bt[b, :-(-n // 16)] = rng.integers(0, pool, size=-(-n // 16))
    par = np.array([-1] + [(i - 1) // 2 for i in range(1, T)], np.int32)
    return dict(dtype=dt, q=mk(B, T, Hq, D), k_cache=mk(pool, Hkv, 16, D), v_cache=mk(pool, Hkv, 16, D), block_table=bt,
                ctx_len=np.array(lens, np.int32), k_tree=mk(B, T, Hkv, D), v_tree=mk(B, T, Hkv, D),
                parents=np.tile(par, (B, 1)), scale=D ** -0.5)


def _call_ws(inp, size, shift=0):
    """The C call with a workspace of size bytes, shift bytes past an aligned address (None:
    sr_tree_verify_attn_noalloc): status, out, lse. Asserts that nothing around the workspace is written, nor the
    workspace itself when it is not aligned."""
    import ctypes as C
    from paper_2608_04962_amd import _lib
    keys = ("q", "k_cache", "v_cache", "block_table", "ctx_len", "k_tree", "v_tree", "parents")
    t = {k: dev_tensor(inp[k]) for k in keys}
    desc = sr.attn_desc(t["q"], t["k_cache"], t["block_table"], inp["scale"])
    out = torch.full(tuple(t["q"].shape), 7.0, device="cuda")
    lse = torch.full(tuple(t["q"].shape[:3]), 7.0, device="cuda")
    args = [C.byref(desc)] + [t[k].data_ptr() for k in keys] + [out.data_ptr(), lse.data_ptr()]
    if size is None:
        st = _lib.lib().sr_tree_verify_attn_noalloc(*args, None)
    else:
        ws = torch.full((256 + shift + size + 4096,), 0xAB, dtype=torch.uint8, device="cuda")
        st = _lib.lib().sr_tree_verify_attn(*args, ws.data_ptr() + 256 + shift if size else None, size, None)
        free = ws[256 + size:] if shift == 0 else ws
        assert bool((free == 0xAB).all()) and bool((ws[:256] == 0xAB).all())
    torch.cuda.synchronize()
    return st, out.cpu().numpy(), lse.cpu().numpy()


def _check_nodes(inp, out, lse, nodes):
    ro, rl = _oracle(inp, nodes)
    sel = ~np.isnan(ro[..., 0])
    assert np.isfinite(out).all()
    assert row_rel_err(out[sel], ro[sel]).max() <= tol_for(inp["dtype"])
    assert np.abs(lse[sel] - rl[sel]).max() <= tol_for(inp["dtype"])


@pytest.mark.parametrize("dt,B,T,G,D,max_blocks,wide", [
    ("f32", 64, 8, 4, 64, 8192, False),        # 512 units: the least workspace of tables wider than the page-id table
    ("bf16", 64, 8, 4, 64, 8192, True),        # the same, with V that is recomputed in fp32
    ("f32", 1, 8, 4, 128, 512, False),         # one unit of 16 chunks
    ("bf16", 3, 8, 2, 128, 700, True),
])
def test_least_workspace_of_long_tables(dt, B, T, G, D, max_blocks, wide):
    """The least workspace with few query rows and many chunks: a segment longer than the page-id table is never made,
    also for contexts past 65536 keys, and no scratch is used past the workspace's end."""
    Hkv = 8 if B == 64 else 1
    top = max_blocks * 16
    lens = [top, top - 15, top * 5 // 8 + 3] + [(37 * b) % 500 for b in range(B)]
    inp = _pooled_inputs(dt, B, T, Hkv * G, Hkv, D, lens[:B], max_blocks, 40, seed=41)
    if wide:
        inp["v_cache"] = synth.as_dtype((synth.to_f64(inp["v_cache"], dt) * 1e5).astype(np.float32), dt)
        inp["v_tree"] = synth.as_dtype((synth.to_f64(inp["v_tree"], dt) * 1e5).astype(np.float32), dt)
    units = B * Hkv
    nch = -(-max_blocks // (32 if units < 64 else 256))
    rows = units * nch * (-(-T * G // 32) * 32)
    up = lambda x: -(-x // 256) * 256
    size = up(rows * D * 4) + up(rows * 8) + (up((3 + 2 * units * nch) * 4) if dt == "bf16" else 0)
    st, out, lse = _call_ws(inp, size)
    assert st == 0
    _check_nodes(inp, out, lse, [(b, u) for b in sorted({0, B // 2, B - 1, min(1, B - 1)}) for u in (0, T - 1)])
    st, _, _ = _call_ws(inp, size - 256)
    assert st == 3                              # SR_ERR_WORKSPACE


def test_noalloc_least_scratch_of_long_tables():
    """sr_tree_verify_attn_noalloc where only the least scratch fits its array, with a context past 65536 keys."""
    B, T, Hkv, G, D, mb = 64, 8, 8, 4, 64, 15872
    lens = [mb * 16, 70001, 65537] + [(53 * b) % 700 for b in range(B)]
    inp = _pooled_inputs("f32", B, T, Hkv * G, Hkv, D, lens[:B], mb, 24, seed=42)
    st, out, lse = _call_ws(inp, None)
    assert st == 0
    _check_nodes(inp, out, lse, [(b, u) for b in (0, 1, 2, 3, 63) for u in (0, T - 1)])


def test_workspace_that_is_not_aligned():
    """fp32 prefixes of one chunk need no workspace and take any: one that is not aligned is left alone. Calls that
    need one refuse it."""
    inp = _pooled_inputs("f32", 3, 8, 8, 4, 64, [500, 0, 317], 32, 40, seed=43)
    st, want, wl = _call_ws(inp, 0)
    assert st == 0
    for shift in (4, 16, 128):
        st, out, lse = _call_ws(inp, 4 << 20, shift)
        assert st == 0
        assert np.array_equal(out, want) and np.array_equal(lse, wl)
    _check_nodes(inp, want, wl, [(b, u) for b in range(3) for u in range(8)])
    inp = _pooled_inputs("f32", 3, 8, 8, 4, 64, [500, 0, 317], 80, 40, seed=43)
    assert _call_ws(inp, 4 << 20, 64)[0] == 1   # SR_ERR_INVALID


def test_python_takes_the_least_workspace():
    """tree_verify_attn takes a workspace that the call takes, smaller than the query's answer; a smaller one still is
    a ValueError. A prefix of one chunk takes any."""
    for lens, mb, rows in (([3000, 17, 900, 4096], 256, 16 * 8 * 32), ([500, 0, 317, 31], 32, 0)):
        inp = _pooled_inputs("f32", 4, 8, 16, 4, 128, lens, mb, 40, seed=44)
        t = {k: dev_tensor(v) for k, v in inp.items() if isinstance(v, np.ndarray)}
        size = rows * (128 + 2) * 4             # 16 units, 32 rows each, a chunk per 32 pages
        assert size < sr.attn_workspace_bytes(sr.attn_desc(t["q"], t["k_cache"], t["block_table"]))

        def call(n):
            return sr.tree_verify_attn(t["q"], t["k_cache"], t["v_cache"], t["block_table"], t["ctx_len"], t["k_tree"],
                                       t["v_tree"], t["parents"], workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))
        out, lse = call(size)
        _check_nodes(inp, out.cpu().numpy(), lse.cpu().numpy(), [(b, u) for b in range(4) for u in (0, 7)])
        if size:
            with pytest.raises(ValueError, match="workspace"):
                call(size - 256)


@pytest.mark.parametrize("dt,B,Hkv,G,T,D,pages", [
    ("bf16", 64, 4, 7, 8, 128, 92), ("bf16", 64, 4, 7, 8, 128, 93),      # 256 units of 24 and 25 tiles
    ("bf16", 32, 4, 2, 65, 64, 48), ("bf16", 257, 1, 4, 5, 128, 24),     # two tree tiles; one unit past the blocks
    ("bf16", 43, 8, 8, 25, 128, 100), ("bf16", 43, 8, 8, 25, 128, 101),  # 344 units of 26 and 27 tiles, dealt and cut
    ("bf16", 512, 1, 3, 4, 64, 30), ("bf16", 11, 8, 5, 96, 128, 40),     # two for every block; three row groups each
    ("bf16", 1, 1, 3, 9, 128, 12), ("f32", 64, 4, 4, 9, 64, 20), ("f32", 64, 4, 8, 9, 128, 20), ("f32", 3, 2, 5, 7, 64, 12)])
def test_units_left_whole(dt, B, Hkv, G, T, D, pages):
    """Short units that are not cut, a block for each or ranges of them, at the rule's line and one past it: contexts of
    no key, one and the table's width, and trajectories with bad lengths and pages."""
    rng = np.random.default_rng(pages)
    lens = [int(x) for x in rng.integers(0, pages * 16 + 1, size=B)]
    lens[0] = pages * 16
    if B > 4:
        lens[1], lens[2], lens[B - 1] = 0, 1, pages * 16
    inp = _pooled_inputs(dt, B, T, Hkv * G, Hkv, D, lens, pages, 50, seed=pages)
    if B > 8:
        inp["ctx_len"][4] = pages * 16 + 1
        inp["ctx_len"][5] = -3
        inp["ctx_len"][6] = max(17, int(inp["ctx_len"][6]))
        inp["block_table"][6, 1] = 50
    t = {k: dev_tensor(v) for k, v in inp.items() if isinstance(v, np.ndarray)}
    out, lse = sr.tree_verify_attn(t["q"], t["k_cache"], t["v_cache"], t["block_table"], t["ctx_len"], t["k_tree"],
                                   t["v_tree"], t["parents"])
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    bad = {4, 5, 6} if B > 8 else set()
    good = [b for b in range(B) if b not in bad]
    for b in bad:
        assert np.isnan(out[b]).all() and np.isnan(lse[b]).all()
    nodes = [(b, u) for b in good[:6] + good[-6:] for u in range(T)]
    ro, rl = _oracle(inp, nodes)
    sel = ~np.isnan(ro[..., 0])
    assert np.isfinite(out[good]).all()
    assert row_rel_err(out[sel], ro[sel]).max() <= tol_for(dt)
    assert np.abs(lse[sel] - rl[sel]).max() <= tol_for(dt)


@pytest.mark.parametrize("dt,wide", [("f32", False), ("bf16", False), ("bf16", True)])
def test_rounds_of_ranges(dt, wide):
    """More tiles than the blocks' page-id tables hold at once: every block takes two ranges, one after the other."""
    B, T, Hkv, G, D, mb = 66, 8, 8, 2, 64, 2048
    lens = [mb * 16 - 7 * b for b in range(B)]
    lens[7] = 5                                  # and a short one among them
    inp = _pooled_inputs(dt, B, T, Hkv * G, Hkv, D, lens, mb, 30, seed=46)
    assert sum(-(-n // 64) + 1 for n in lens) * Hkv > 256 * 1024
    if wide:
        inp["v_tree"][5:9] = synth.as_dtype((synth.to_f64(inp["v_tree"][5:9], dt) * 1e6).astype(np.float32), dt)
    t = {k: dev_tensor(v) for k, v in inp.items() if isinstance(v, np.ndarray)}
    out, lse = sr.tree_verify_attn(t["q"], t["k_cache"], t["v_cache"], t["block_table"], t["ctx_len"], t["k_tree"],
                                   t["v_tree"], t["parents"])
    _check_nodes(inp, out.cpu().numpy(), lse.cpu().numpy(), [(b, u) for b in (0, 7, 8, 33, 64, 65) for u in (0, T - 1)])


def test_cut_of_lognormal_contexts():
    """256 trajectories of lognormal contexts with few rows: many units cut by the ranges of the 256 blocks."""
    rng = np.random.default_rng(47)
    lens = [int(x) for x in np.clip(np.exp(np.log(1000) + rng.standard_normal(256)), 1, 8192)]
    inp = _pooled_inputs("bf16", 256, 8, 14, 2, 128, lens, 512, 60, seed=47)
    t = {k: dev_tensor(v) for k, v in inp.items() if isinstance(v, np.ndarray)}
    out, lse = sr.tree_verify_attn(t["q"], t["k_cache"], t["v_cache"], t["block_table"], t["ctx_len"], t["k_tree"],
                                   t["v_tree"], t["parents"])
    _check_nodes(inp, out.cpu().numpy(), lse.cpu().numpy(), [(b, u) for b in range(0, 256, 5) for u in (0, 7)])


def test_dealt_units_with_wide_values():
    """Units dealt to the blocks by length, some with V outside fp16's range (recomputed in the block) and ties among
    the lengths."""
    lens = [int(x) for x in np.random.default_rng(48).choice([1, 64, 65, 500, 501, 900], size=100)]
    inp = _pooled_inputs("bf16", 100, 6, 12, 3, 128, lens, 60, 64, seed=48)
    vt = synth.to_f64(inp["v_tree"], "bf16")
    vt[::7] *= 1e6
    inp["v_tree"] = synth.as_dtype(vt.astype(np.float32), "bf16")
    t = {k: dev_tensor(v) for k, v in inp.items() if isinstance(v, np.ndarray)}
    call = lambda: sr.tree_verify_attn(t["q"], t["k_cache"], t["v_cache"], t["block_table"], t["ctx_len"], t["k_tree"],
                                       t["v_tree"], t["parents"])
    out, lse = call()
    out2, lse2 = call()
    assert torch.equal(out, out2) and torch.equal(lse, lse2)
    _check_nodes(inp, out.cpu().numpy(), lse.cpu().numpy(), [(b, u) for b in range(100) for u in (0, 2, 5)])
