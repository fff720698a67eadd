"""GPU parity of cf_decode_layer (RMSNorm in front of the block, residual connection behind it, fused into the
same kernel) against the CPU oracle's decode_layer, through the C ABI.

Tolerance: that of the block (max|err| <= 1e-2 * max|ref| + 1e-3 on the output plus the stage-wise checks of
test_gpu_parity.check).  The mean square of a row is a fp32 sum of D squares (relative error ~1e-7), far
inside the stage-wise bound of 2e-5 on the rotated queries.
"""
import numpy as np
import pytest

import cf_inputs
import plan_arith
from oracle import decode_block as orc
from oracle import c_oracle
from test_gpu_parity import check, _log

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def gamma_for(shape, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return (1.0 + 0.25 * rng.standard_normal(shape.d_model)).astype(np.float16)


def run_layer(shape, batch, inp, pos, gamma, eps, residual, packed):
    from paper_2508_18850_amd import DecodeBlock
    dev = torch.device("cuda:0")
    blk = DecodeBlock(shape.d_model, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, batch, inp["max_seq"],
                      shape.rope_base, debug=True)
    st = torch.cuda.current_stream().cuda_stream
    t = {k: torch.from_numpy(inp[k]).to(dev) for k in ("x", "w_qkv", "w_o", "k_cache", "v_cache")}
    g = torch.from_numpy(gamma).to(dev) if gamma is not None else None
    out = torch.full((batch, shape.d_model), float("nan"), dtype=torch.float16, device=dev)
    wq, wo = t["w_qkv"], t["w_o"]
    if packed:
        nq_bytes, no_bytes = blk.packed_sizes()
        wq = torch.empty((nq_bytes // 2,), dtype=torch.float16, device=dev)
        wo = torch.empty((no_bytes // 2,), dtype=torch.float16, device=dev)
        blk.pack_weights(t["w_qkv"].data_ptr(), t["w_o"].data_ptr(), wq.data_ptr(), wo.data_ptr(), st)
    blk.decode_layer(batch, t["x"].data_ptr(), g.data_ptr() if g is not None else 0, eps, residual, packed,
                     wq.data_ptr(), wo.data_ptr(), t["k_cache"].data_ptr(), t["v_cache"].data_ptr(), pos,
                     out.data_ptr(), st)
    blk.status(st)
    res = {"out": out.cpu().numpy(), "k_cache": t["k_cache"].cpu().numpy(), "v_cache": t["v_cache"].cpu().numpy()}
    for what, key in ((0, "q_rot"), (1, "attn")):
        a = np.empty((batch, shape.n_q_heads, shape.head_dim), dtype=np.float32)
        blk.debug_export(what, a, st)
        res[key] = a
    assert np.array_equal(t["x"].cpu().numpy().view(np.uint16), inp["x"].view(np.uint16)), "x was modified"
    blk.close()
    return res


def reference(shape, inp, pos, gamma, eps, residual, use_c=False):
    args = (inp["w_qkv"], inp["w_o"], inp["k_cache"], inp["v_cache"], pos, shape.n_q_heads, shape.n_kv_heads,
            shape.head_dim, shape.rope_base)
    if gamma is None:
        ref = (c_oracle.decode_block if use_c else orc.decode_block)(inp["x"], *args)
        if residual:
            ref["out"] = ref["out"] + inp["x"].astype(np.float64)
        return ref
    ref = (c_oracle.decode_layer if use_c else orc.decode_layer)(inp["x"], gamma, eps, *args)
    if not residual:
        ref["out"] = ref["out"] - inp["x"].astype(np.float64)
    return ref


SHAPES = [
    ("tiny", cf_inputs.SHAPES["tiny"], 1, 256),
    ("ragged_d64_g2_b3", cf_inputs.BlockShape("small", 264, 4, 2, 64, 10000.0, 77), 3, 77),
    ("d128_g4_b4", cf_inputs.BlockShape("s", 1024, 16, 4, 128, 500000.0, 333), 4, 333),
    ("d128_g1_b16", cf_inputs.BlockShape("s", 512, 8, 8, 128, 10000.0, 130), 16, 130),
    ("d128_g8_b5", cf_inputs.BlockShape("s", 2048, 16, 2, 128, 10000.0, 45), 5, 45),
]


@pytest.mark.parametrize("name,shape,batch,kv_len", SHAPES)
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("norm,residual", [(True, True), (True, False), (False, True)])
def test_layer_matches_oracle(name, shape, batch, kv_len, packed, norm, residual):
    _log("layer case %s B=%d L=%d packed=%s norm=%s residual=%s" % (name, batch, kv_len, packed, norm, residual))
    inp = cf_inputs.make_inputs(shape, seed=23, batch=batch, kv_len=kv_len)
    # rows of different scale, so that a wrong or shared normalisation factor shows
    scale = np.array([0.25 * (b + 1) for b in range(batch)], dtype=np.float32)[:, None]
    inp["x"] = (inp["x"].astype(np.float32) * scale).astype(np.float16)
    gamma = gamma_for(shape, 5) if norm else None
    eps = 1e-5
    res = run_layer(shape, batch, inp, kv_len, gamma, eps, residual, packed)
    check(res, reference(shape, inp, kv_len, gamma, eps, residual), inp, kv_len, name)


def test_large_eps_and_zero_row():
    # a zero row normalises to zero (eps keeps the factor finite); a large eps changes the factor visibly
    shape, batch, kv_len = cf_inputs.BlockShape("s", 512, 8, 2, 64, 10000.0, 50), 2, 50
    inp = cf_inputs.make_inputs(shape, seed=3, batch=batch, kv_len=kv_len)
    inp["x"][1] = 0
    gamma = gamma_for(shape, 6)
    for eps in (1e-6, 0.5):
        res = run_layer(shape, batch, inp, kv_len, gamma, eps, True, True)
        check(res, reference(shape, inp, kv_len, gamma, eps, True), inp, kv_len, "eps=%g" % eps)


@pytest.mark.parametrize("workload,batch", [("llama2_7b", 1), ("llama3_8b", 4)])
def test_full_size_layer(workload, batch):
    """The configuration the bench times (packed weights), with normalisation and residual, against the C oracle."""
    shape = cf_inputs.SHAPES[workload]
    _log("full-size layer %s B=%d" % (workload, batch))
    inp = cf_inputs.make_inputs(shape, seed=1000, batch=batch)
    gamma = gamma_for(shape, 7)
    res = run_layer(shape, batch, inp, shape.kv_len, gamma, 1e-5, True, True)
    check(res, reference(shape, inp, shape.kv_len, gamma, 1e-5, True, use_c=True), inp, shape.kv_len, workload)


def test_layer_arguments_are_checked():
    from paper_2508_18850_amd import DecodeBlock
    shape = cf_inputs.SHAPES["tiny"]
    blk = DecodeBlock(shape.d_model, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, 1, 64, shape.rope_base)
    a = torch.zeros(1 << 20, dtype=torch.float16, device="cuda")
    p = a.data_ptr()
    assert blk.decode_layer_rc(1, p, p, -1.0, 1, 0, p, p, p, p, 3, p + 4096) == -1            # negative eps
    assert blk.decode_layer_rc(1, p, p, float("nan"), 1, 0, p, p, p, p, 3, p + 4096) == -1    # eps not a number
    assert blk.decode_layer_rc(1, p, p + 2, 1e-5, 1, 0, p, p, p, p, 3, p + 4096) == -1        # misaligned weight
    assert blk.decode_layer_rc(1, p, p, 1e-5, 1, 0, p, p, p, p, 3, p) == -1                   # out == x with residual
    blk.close()


# ---------------------------------------------------------------------------------------------------
# rows with positions of their own (cf_decode_layer_rows)
# ---------------------------------------------------------------------------------------------------

def run_rows(shape, batch, inp, row_pos, max_pos, gamma, eps, residual, packed, kv_splits=0):
    from paper_2508_18850_amd import DecodeBlock
    dev = torch.device("cuda:0")
    blk = DecodeBlock(shape.d_model, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, batch, inp["max_seq"],
                      shape.rope_base, debug=True)
    if kv_splits:
        blk.set_tuning(kv_splits=kv_splits)
    st = torch.cuda.current_stream().cuda_stream
    t = {k: torch.from_numpy(inp[k]).to(dev) for k in ("x", "w_qkv", "w_o", "k_cache", "v_cache")}
    g = torch.from_numpy(gamma).to(dev) if gamma is not None else None
    rp = torch.tensor(list(row_pos), dtype=torch.int32, device=dev)
    out = torch.full((batch, shape.d_model), float("nan"), dtype=torch.float16, device=dev)
    wq, wo = t["w_qkv"], t["w_o"]
    if packed:
        nq_bytes, no_bytes = blk.packed_sizes()
        wq = torch.empty((nq_bytes // 2,), dtype=torch.float16, device=dev)
        wo = torch.empty((no_bytes // 2,), dtype=torch.float16, device=dev)
        blk.pack_weights(t["w_qkv"].data_ptr(), t["w_o"].data_ptr(), wq.data_ptr(), wo.data_ptr(), st)
    blk.decode_layer_rows(batch, t["x"].data_ptr(), g.data_ptr() if g is not None else 0, eps, residual, packed,
                          wq.data_ptr(), wo.data_ptr(), t["k_cache"].data_ptr(), t["v_cache"].data_ptr(),
                          rp.data_ptr(), max_pos, out.data_ptr(), st)
    blk.status(st)
    res = {"out": out.cpu().numpy(), "k_cache": t["k_cache"].cpu().numpy(), "v_cache": t["v_cache"].cpu().numpy()}
    for what, key in ((0, "q_rot"), (1, "attn")):
        a = np.empty((batch, shape.n_q_heads, shape.head_dim), dtype=np.float32)
        blk.debug_export(what, a, st)
        res[key] = a
    plan = blk.plan()
    _log("plan %s" % plan)
    blk.close()
    res["plan"] = plan
    return res


def check_rows(res, ref, inp, row_pos, label):
    """test_gpu_parity.check row by row (each row has its own appended cache row)."""
    for b, pos in enumerate(row_pos):
        one = {k: v[b:b + 1] for k, v in res.items() if k != "plan"}
        refb = {k: v[b:b + 1] for k, v in ref.items()}
        inpb = {k: inp[k][b:b + 1] for k in ("k_cache", "v_cache")}
        check(one, refb, inpb, pos, "%s row %d pos %d" % (label, b, pos))


ROW_CASES = [
    # name, shape, positions of the rows (capacity = max + a few rows)
    ("d64_g2", cf_inputs.BlockShape("small", 264, 4, 2, 64, 10000.0, 77), [77, 0, 5]),
    ("d128_g4", cf_inputs.BlockShape("s", 1024, 16, 4, 128, 500000.0, 333), [1, 333, 332, 100]),
    ("d128_g1_b16", cf_inputs.BlockShape("s", 512, 8, 8, 128, 10000.0, 130),
     [130, 129, 1, 0, 64, 65, 33, 32, 31, 2, 100, 17, 130, 77, 3, 128]),
    ("d128_g8_b2", cf_inputs.BlockShape("s", 2048, 16, 2, 128, 10000.0, 1000), [1000, 250]),
    ("d128_g1_b1", cf_inputs.BlockShape("s", 512, 8, 8, 128, 10000.0, 300), [123]),      # bound above the only row
]


@pytest.mark.parametrize("name,shape,row_pos", ROW_CASES)
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("layer", [True, False])
def test_rows_with_own_positions_match_oracle(name, shape, row_pos, packed, layer):
    batch, max_pos = len(row_pos), shape.kv_len
    _log("rows case %s pos=%s packed=%s layer=%s" % (name, row_pos, packed, layer))
    inp = cf_inputs.make_inputs(shape, seed=31, batch=batch, kv_len=max_pos)
    # cached rows at and beyond a row's own position must never be read: poison them
    for b, pos in enumerate(row_pos):
        inp["k_cache"][b, :, pos:] = np.nan
        inp["v_cache"][b, :, pos:] = np.nan
    gamma = gamma_for(shape, 9) if layer else None
    res = run_rows(shape, batch, inp, row_pos, max_pos, gamma, 1e-5, layer, packed)
    ref = orc.decode_rows(inp["x"], gamma, 1e-5, inp["w_qkv"], inp["w_o"], inp["k_cache"], inp["v_cache"], row_pos,
                          shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rope_base)
    check_rows(res, ref, inp, row_pos, name)


# Lengths so far apart that the kernel deals the attention items by them: every batch tile and width of the merge (values per
# thread), more than 32 splits of a row, rows without a token, all rows shorter than the bound, as many members as rows and one more.
DEALT = [
    ("d128_g4_b4", cf_inputs.BlockShape("s", 512, 8, 2, 128, 10000.0, 52000), [3000, 5, 0, 700]),
    ("d128_g1_b1", cf_inputs.BlockShape("s", 256, 32, 32, 128, 10000.0, 9000), [1000]),
    ("d128_g2_b2", cf_inputs.BlockShape("s", 264, 2, 1, 128, 10000.0, 25000), [6000, 40]),
    ("d128_g1_b9", cf_inputs.BlockShape("s", 512, 8, 8, 128, 500000.0, 2100), [2100, 1, 2, 3, 400, 0, 31, 32, 33]),
    ("d128_g8_b16", cf_inputs.BlockShape("s", 264, 32, 4, 128, 10000.0, 2000), [2000] + [17 * b for b in range(15)]),
    ("d128_g1_b16_17_members", cf_inputs.BlockShape("s", 264, 15, 15, 128, 10000.0, 1500), [40] * 15 + [1500]),
    ("d64_g1_b5", cf_inputs.BlockShape("s", 520, 16, 16, 64, 10000.0, 4000), [4000, 10, 20, 30, 3999]),
    ("d64_g2_b3", cf_inputs.BlockShape("s", 520, 16, 8, 64, 10000.0, 6500), [64, 6500, 65]),
    ("d64_g8_b2", cf_inputs.BlockShape("s", 520, 16, 2, 64, 10000.0, 60000), [0, 0]),
    ("d64_g1_b16_16_members", cf_inputs.BlockShape("s", 520, 16, 16, 64, 10000.0, 2000), [1000] + [60 * b for b in range(15)]),
    ("d128_g1_b8_8_members", cf_inputs.BlockShape("s", 256, 32, 32, 128, 10000.0, 1500), [700, 0, 3, 699, 500, 31, 257, 1]),
]


def dealt_inputs(shape, row_pos):
    inp = cf_inputs.make_inputs(shape, seed=33, batch=len(row_pos), kv_len=max(row_pos))
    for b, pos in enumerate(row_pos):                       # rows at and beyond a row's position are never read
        inp["k_cache"][b, :, pos:] = np.nan
        inp["v_cache"][b, :, pos:] = np.nan
    # the bound is an argument of the plan; the caches have to hold it
    grow = shape.kv_len + 1 - inp["max_seq"]
    if grow > 0:
        for c in ("k_cache", "v_cache"):
            inp[c] = np.concatenate([inp[c], np.full(inp[c].shape[:2] + (grow, shape.head_dim), np.nan, dtype=np.float16)], axis=2)
        inp["max_seq"] = shape.kv_len + 1
    return inp


@pytest.mark.parametrize("name,shape,row_pos", DEALT)
def test_rows_of_very_different_lengths(name, shape, row_pos):
    _log("dealt rows case %s pos=%s" % (name, row_pos))
    batch, max_pos = len(row_pos), shape.kv_len
    inp = dealt_inputs(shape, row_pos)
    gamma = gamma_for(shape, 11)
    res = run_rows(shape, batch, inp, row_pos, max_pos, gamma, 1e-5, True, True)
    ref = orc.decode_rows(inp["x"], gamma, 1e-5, inp["w_qkv"], inp["w_o"], inp["k_cache"], inp["v_cache"], row_pos,
                          shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rope_base)
    check_rows(res, ref, inp, row_pos, name)


# Both sides of the gain from which items are dealt: two rows of 6000 and 4800 tokens over eight members take 1500 tokens a member,
# the plan for a bound of 6316 / 6320 tokens 1595 / 1596, and the gain asked for is 96.
NEARLY = [("d128_g1_b2_%s" % ("dealt" if bound == 6320 else "planned"), cf_inputs.BlockShape("s", 256, 32, 32, 128, 10000.0, bound), [6000, 4800])
          for bound in (6316, 6320)]


@pytest.mark.parametrize("name,shape,row_pos", DEALT + NEARLY)
def test_dealt_items_are_the_ones_that_run(name, shape, row_pos):
    """Which items ran shows in the bits of the attention result, since the partials of other splits add up to other bits: with items
    dealt into two and more splits of a row they are not those of the plan's splits (which a call with tuned splits takes), otherwise they
    are.  Two calls with the same lengths give the same bits."""
    _log("dealt items case %s pos=%s" % (name, row_pos))
    inp = dealt_inputs(shape, row_pos)
    gamma = gamma_for(shape, 11)
    args = (shape, len(row_pos), inp, row_pos, shape.kv_len, gamma, 1e-5, True, True)
    res, again = run_rows(*args), run_rows(*args)
    for key in ("attn", "q_rot", "out", "k_cache", "v_cache"):
        assert res[key].tobytes() == again[key].tobytes(), key
    plan, gain = res["plan"], plan_arith.ragged_gain(shape.head_dim)
    assert plan["tokens_per_split"] >= 4 * gain, plan
    d = plan_arith.deal(row_pos, plan["team_size"], plan["tokens_per_split"], gain,
                        int(plan["team_size"] % 2 == 0 and plan["workgroups"] % 2 == 0))
    assert (d.items > 0) == (not name.endswith("planned")), (plan, d)
    planned = run_rows(*args, kv_splits=plan["kv_splits"])
    assert all(planned["plan"][k] == plan[k] for k in ("kv_splits", "tokens_per_split", "team_size")), planned["plan"]
    same = planned["attn"].tobytes() == res["attn"].tobytes()
    _log("   %d items of %d tokens, splits %s, same bits as the plan's: %s" % (d.items, d.size, d.splits, same))
    if d.items == 0:
        assert same
    elif max(d.splits) > 1:
        assert not same


def test_rows_when_a_workgroup_handles_several_rows():
    """More (row, split) items than workgroups in a team: a workgroup goes from one row to another and has to
    rebuild its RoPE table for the other row's position."""
    shape = cf_inputs.BlockShape("s", 512, 8, 8, 128, 10000.0, 130)
    row_pos = [130, 129, 1, 0, 64, 65, 33, 32, 31, 2, 100, 17, 130, 77, 3, 128]
    inp = cf_inputs.make_inputs(shape, seed=32, batch=16, kv_len=130)
    gamma = gamma_for(shape, 10)
    res = run_rows(shape, 16, inp, row_pos, 130, gamma, 1e-5, True, True, kv_splits=4)
    assert 16 * res["plan"]["kv_splits"] > res["plan"]["team_size"], res["plan"]
    ref = orc.decode_rows(inp["x"], gamma, 1e-5, inp["w_qkv"], inp["w_o"], inp["k_cache"], inp["v_cache"], row_pos,
                          shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rope_base)
    check_rows(res, ref, inp, row_pos, "several rows per workgroup")


def test_full_size_rows():
    """Llama-3-8B shape, four rows of different lengths (packed weights), against the C oracle row by row."""
    shape = cf_inputs.SHAPES["llama3_8b"]
    row_pos = [shape.kv_len, shape.kv_len // 2 + 3, 17, shape.kv_len - 1]
    inp = cf_inputs.make_inputs(shape, seed=1001, batch=4)
    for b, pos in enumerate(row_pos):
        inp["k_cache"][b, :, pos:] = np.nan
        inp["v_cache"][b, :, pos:] = np.nan
    gamma = gamma_for(shape, 8)
    res = run_rows(shape, 4, inp, row_pos, shape.kv_len, gamma, 1e-5, True, True)
    ref = orc.decode_rows(inp["x"], gamma, 1e-5, inp["w_qkv"], inp["w_o"], inp["k_cache"], inp["v_cache"], row_pos,
                          shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rope_base,
                          layer_fn=c_oracle.decode_layer, block_fn=c_oracle.decode_block)
    check_rows(res, ref, inp, row_pos, "llama3_8b rows")


def test_row_positions_outside_the_bound_are_clamped():
    # an entry above max_pos is read as max_pos, a negative one as 0: the kernel stays inside its buffers
    shape = cf_inputs.BlockShape("s", 512, 8, 2, 64, 10000.0, 40)
    inp = cf_inputs.make_inputs(shape, seed=4, batch=2, kv_len=40)
    res = run_rows(shape, 2, inp, [10 ** 6, -5], 40, None, 0.0, False, False)
    ref = orc.decode_rows(inp["x"], None, 0.0, inp["w_qkv"], inp["w_o"], inp["k_cache"], inp["v_cache"], [40, 0],
                          shape.n_q_heads, shape.n_kv_heads, shape.head_dim, shape.rope_base)
    check_rows(res, ref, inp, [40, 0], "clamped")


# Slices that do not come out even, with the row norms of every batch tile: rows of more than 4096 values (two loads per
# thread), batches that take a second group of rows (more than eight), slices staged in pieces of eight values.
@pytest.mark.parametrize("d_model,nq,nkv,hd,batch", [(1000, 32, 8, 128, 1), (1000, 32, 8, 128, 3), (1032, 8, 8, 128, 9),
                                                     (1032, 8, 8, 128, 16), (4104, 8, 4, 128, 10), (1288, 14, 7, 64, 2),
                                                     (1288, 14, 7, 64, 16), (8192, 4, 4, 128, 1)])
def test_layer_with_uneven_slices(d_model, nq, nkv, hd, batch):
    shape, kv_len = cf_inputs.BlockShape("s", d_model, nq, nkv, hd, 10000.0, 60), 60
    _log("layer d_model %d heads %d/%d x %d batch %d" % (d_model, nq, nkv, hd, batch))
    inp = cf_inputs.make_inputs(shape, seed=29, batch=batch, kv_len=kv_len)
    scale = np.array([0.25 * (b + 1) for b in range(batch)], dtype=np.float32)[:, None]
    inp["x"] = (inp["x"].astype(np.float32) * scale).astype(np.float16)
    gamma = gamma_for(shape, 9)
    res = run_layer(shape, batch, inp, kv_len, gamma, 1e-5, True, True)
    check(res, reference(shape, inp, kv_len, gamma, 1e-5, True), inp, kv_len, "uneven")


# Slices of 33 rows, not a multiple of eight: x (and the norm's weights) staged value by value.
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("hd,batch", [(128, 1), (128, 2), (128, 9), (128, 16), (64, 3), (64, 16)])
def test_slices_that_are_no_multiple_of_eight_rows(hd, batch, norm, monkeypatch):
    import paper_2508_18850_amd as cf

    class Tuned(cf.DecodeBlock):
        def __init__(self, *args, **kwargs):
            super().__init__(*args, **kwargs)
            self.set_tuning(k_splits=32)

        def close(self):
            assert self.plan()["rows_per_split"] == 33
            super().close()

    monkeypatch.setattr(cf, "DecodeBlock", Tuned)
    shape, kv_len = cf_inputs.BlockShape("s", 1032, 8, 8, hd, 10000.0, 40), 40
    _log("33-row slices, head_dim %d batch %d norm %s" % (hd, batch, norm))
    inp = cf_inputs.make_inputs(shape, seed=31, batch=batch, kv_len=kv_len)
    gamma = gamma_for(shape, 10) if norm else None
    res = run_layer(shape, batch, inp, kv_len, gamma, 1e-5, norm, True)
    check(res, reference(shape, inp, kv_len, gamma, 1e-5, norm), inp, kv_len, "33 rows")


# Operands of the two projections far from one, their counterparts scaled the other way (powers of two on the inputs): x * gamma
# at 4e-6, up to 1e5 and up to 8e6 (fp16 ends at 65504), rows of one batch 2^16 apart, attention outputs at 1e-6.
MAGNITUDES = {
    "small x gamma": dict(x=-8, gamma=-10, w_qkv=10),
    "large x gamma": dict(x=13, gamma=2, w_qkv=-2),
    "largest x gamma": dict(x=13, gamma=8, w_qkv=-8),
    "rows apart": dict(rows=True),
    "small attention output": dict(w_v=-10, v_cache=-20, w_o=12),
}


@pytest.mark.parametrize("d_model,hd,batch,tuning", [
    (520, 64, 1, {}), (520, 64, 5, {}), (520, 64, 16, {}), (520, 128, 1, {}), (520, 128, 5, {}), (520, 128, 16, {}),
    (520, 64, 7, dict(k_splits=16)), (520, 128, 16, dict(k_splits=16)),         # slices of 33 rows, staged value by value
    (1320, 64, 16, dict(workgroups=4)), (1320, 128, 9, dict(workgroups=4)),     # slices of 1320 rows: more than 32 x 4 pieces a row
])
@pytest.mark.parametrize("name", list(MAGNITUDES))
def test_operands_of_any_magnitude(name, d_model, hd, batch, tuning, monkeypatch):
    """The rotated queries are one fp32 sum of d_model terms whose operands are held in full: relative RMS about
    sqrt(d_model) * 2^-24 at most, 1.5 of that allowed, at every magnitude and batch.  Appended rows and output end in fp16
    (relative RMS 2^-12.5), attention is summed in fp32 over 300 rows (1e-4)."""
    import paper_2508_18850_amd as cf

    class Tuned(cf.DecodeBlock):
        def __init__(self, *args, **kwargs):
            super().__init__(*args, **kwargs)
            if tuning:
                self.set_tuning(**tuning)

    monkeypatch.setattr(cf, "DecodeBlock", Tuned)
    shape, kv_len, s = cf_inputs.BlockShape("s", d_model, 8, 4, hd, 10000.0, 300), 300, MAGNITUDES[name]
    inp = cf_inputs.make_inputs(shape, seed=500 + batch, batch=batch, kv_len=kv_len)
    gamma = gamma_for(shape, 11)

    def scaled(a, e):
        return (a.astype(np.float32) * np.float32(2.0) ** e).astype(np.float16)

    for k in ("x", "w_qkv", "v_cache", "w_o"):
        inp[k] = scaled(inp[k], s.get(k, 0))
    gamma = scaled(gamma, s.get("gamma", 0))
    first_v = (shape.n_q_heads + shape.n_kv_heads) * hd
    inp["w_qkv"][:, first_v:] = scaled(inp["w_qkv"][:, first_v:], s.get("w_v", 0))
    if s.get("rows"):
        inp["x"] = scaled(inp["x"], np.array([(5 * b) % 17 - 8 for b in range(batch)], dtype=np.float32)[:, None])
    for norm in (True, False) if "attention" in name else (True,):
        res = run_layer(shape, batch, inp, kv_len, gamma if norm else None, 0.0, False, True)
        ref = reference(shape, inp, kv_len, gamma if norm else None, 0.0, False)
        _log("%s D %d head_dim %d batch %d norm %s: |x gamma| %.1e |attn| %.1e |out| %.1e" % (
            name, d_model, hd, batch, norm, np.abs(inp["x"].astype(np.float64) * gamma.astype(np.float64)).max(),
            np.abs(ref["attn"]).max(), np.abs(ref["out"]).max()))
        for what, got, want, tol in (("q_rot", res["q_rot"], ref["q_rot"], 1.5 * np.sqrt(d_model) * 2.0 ** -24),
                                     ("attn", res["attn"], ref["attn"], 1e-4), ("out", res["out"], ref["out"], 1e-3),
                                     ("k", res["k_cache"][:, :, kv_len], ref["k_rot"], 1e-3),
                                     ("v", res["v_cache"][:, :, kv_len], ref["v_new"], 1e-3)):
            got = got.astype(np.float64)
            rel = np.sqrt(np.mean((got - want) ** 2) / np.mean(want ** 2))
            _log("   %s: relative RMS %.2e" % (what, rel))
            assert np.isfinite(got).all() and rel < tol, what


@pytest.mark.parametrize("d_model,hd,batch", [(1976, 64, 5), (1976, 64, 16), (1392, 128, 3), (1392, 128, 16)])
def test_longest_slices_of_the_layer(d_model, hd, batch, monkeypatch):
    """As many workgroups as KV heads: one slice, about as long as LDS holds with the low parts of x * gamma beside it; a row has more pieces
    than its lanes keep in registers at batch 16."""
    import paper_2508_18850_amd as cf

    class Tuned(cf.DecodeBlock):
        def __init__(self, *args, **kwargs):
            super().__init__(*args, **kwargs)
            self.set_tuning(workgroups=2)

    monkeypatch.setattr(cf, "DecodeBlock", Tuned)
    shape, kv_len = cf_inputs.BlockShape("s", d_model, 2, 2, hd, 10000.0, 40), 40
    inp = cf_inputs.make_inputs(shape, seed=batch, batch=batch, kv_len=kv_len)
    gamma = gamma_for(shape, 12)
    res = run_layer(shape, batch, inp, kv_len, gamma, 1e-5, True, True)
    check(res, reference(shape, inp, kv_len, gamma, 1e-5, True), inp, kv_len, "one slice of %d" % d_model)


@pytest.mark.parametrize("hd,batch", [(64, 4), (64, 5), (128, 16)])
def test_infinite_input_stays_in_its_row(hd, batch):
    """Rows 1 and 2 hold an infinity and a NaN; every other row gives the bits it gives without them."""
    shape, kv_len = cf_inputs.BlockShape("s", 520, 8, 4, hd, 10000.0, 50), 50
    inp = cf_inputs.make_inputs(shape, seed=7, batch=batch, kv_len=kv_len)
    gamma, rows = gamma_for(shape, 3), [b for b in range(batch) if b not in (1, 2)]
    want = run_layer(shape, batch, inp, kv_len, gamma, 1e-5, True, True)
    inp["x"][1, 77], inp["x"][2, 300] = np.inf, np.nan
    got = run_layer(shape, batch, inp, kv_len, gamma, 1e-5, True, True)
    for what in ("out", "k_cache", "v_cache"):
        assert np.array_equal(got[what][rows].view(np.uint16), want[what][rows].view(np.uint16)), what
    assert not np.isfinite(got["out"][1]).any() and not np.isfinite(got["out"][2]).any()
