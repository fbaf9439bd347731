"""Edges of the kernels' tile and dispatch rules against the fp64 oracle.

Each test walks the sizes around one rule (tile remainders, the switch
between two variants, rows that are not 16-byte aligned) and says where its
tolerance comes from.
"""
import numpy as np
import pytest

from gpu_common import (TOL_HDRAFT, TOL_VARIANT, TOL_Z, device_states, make_case, make_predictor, oracle_for, oracle_states, reduced_shape, rel_fro,
                        require_gpu, say, step_inputs, tensor_to_f64, z_errors)

from test_gemm_dispatch import BF16, E4M3, QKV_ROPE, RESID, STORE_F32, SWIGLU, library_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _against_oracle(case, sample, tol_h, tol_z, steps=1):
    """Prefill and `steps` decode steps of a batch; the requests in `sample`
    are recomputed by the oracle."""
    lens = case.lens
    n = len(lens)
    off = np.concatenate([[0], np.cumsum(lens)])
    pred = make_predictor(case, max_seq_len=int(lens.max()) + steps + 16)
    z, h = pred.prefill(list(range(n)), lens, *device_states(case), want_hdraft=True)
    z, h = tensor_to_f64(z), tensor_to_f64(h)
    orc, O = oracle_for(case), oracle_states(case)
    ref = {i: orc.prefill_one(*(x[off[i]:off[i + 1]] for x in O)) for i in sample}
    for i in sample:
        assert rel_fro(h[off[i]:off[i + 1]], ref[i][1]) <= tol_h, i
    assert z_errors(z[list(sample)], [ref[i][0] for i in sample]).max() <= tol_z
    st = {i: ref[i][2] for i in sample}
    for k in range(1, steps + 1):
        arrays = step_inputs(case, k)
        z, h = pred.step(list(range(n)), *device_states(case, arrays), want_hdraft=True)
        z, h = tensor_to_f64(z), tensor_to_f64(h)
        S = oracle_states(case, arrays)
        zr = []
        for i in sample:
            zi, hi = orc.step_one(st[i], *(x[i] for x in S))[:2]
            zr.append(zi)
            assert rel_fro(h[i], np.asarray(hi).reshape(-1)) <= tol_h, (k, i)
        assert z_errors(z[list(sample)], zr).max() <= tol_z
    pred.close()


@pytest.mark.parametrize("tokens", [1, 15, 17, 500, 2100, 9000])
@pytest.mark.parametrize("aligned", [True, False], ids=["16-byte rows", "odd rows"])
def test_fp32_gemm_tile_sizes(tokens, aligned):
    """16, 32 and 64-row tiles, full and ragged, with 16-byte loads and with
    element loads (widths that are not multiples of 16).  Tolerance: fp32
    sums of up to 768 terms through five layers, sqrt(768) * 2^-24 * 5 ~ 8e-6."""
    shape = dict(d=256, n_q=4, n_kv=2, hd=64, ffn=688, head_hidden=128, theta=1e4) if aligned else \
        dict(d=250, n_q=4, n_kv=2, hd=64, ffn=691, head_hidden=130, theta=1e4)
    lens = [min(200, tokens)] * (tokens // 200) + ([tokens % 200] if tokens % 200 else [])
    say(f"case: fp32 layer d={shape['d']}, {tokens} tokens in {len(lens)} requests, 1 step")
    case = make_case(0, lens=lens, shape=reduced_shape(**shape), n_req=len(lens))
    _against_oracle(case, sorted({0, len(lens) // 2, len(lens) - 1}), 1e-5, 1e-5)


@pytest.mark.parametrize("cfg", [1, 4], ids=["bf16", "e4m3"])
@pytest.mark.parametrize("tokens,requests", [(515, 3), (2050, 90), (16500, 620)])
def test_large_tile_gemm_edges(cfg, tokens, requests):
    """256-row tiles: K splits of one and of odd numbers of slices (515 and
    2,050 rows; 620 requests give the head's K split one slice each), the
    unsplit RoPE epilogue with prompts that start anywhere in the tile's
    four-row groups, more tiles than CUs and a ragged last row tile (16,500
    rows).  Tolerance: the repository's bounds for bf16 and e4m3 layers."""
    r = np.random.default_rng(tokens)
    cut = np.sort(r.choice(np.arange(1, tokens), requests - 1, replace=False))
    lens = np.diff(np.concatenate([[0], cut, [tokens]]))
    shape = reduced_shape(d=256, n_q=4, n_kv=2, ffn=640, head_hidden=256)
    say(f"case: 256-row tiles, cfg {cfg}, {tokens} tokens in {requests} requests (longest {lens.max()}), 1 step")
    case = make_case(cfg, lens=lens, shape=shape, n_req=requests)
    sample = sorted({0, int(lens.argmax()), requests // 3, requests // 2, requests - 1})
    _against_oracle(case, sample, TOL_HDRAFT[case.fmt], TOL_Z[case.fmt])


@pytest.mark.parametrize("cfg", [1, 4], ids=["bf16", "e4m3"])
@pytest.mark.parametrize("tokens", [16385, 16500])
def test_k_split_last_round_of_large_tiles(cfg, tokens):
    """The last tiles of a large GEMM as K splits into blocks of their own, and
    their reduce (residual, fp32 and SwiGLU outputs): the last row tile, of
    one and of 116 rows.  Tolerance: the repository's bounds for bf16 and e4m3
    layers."""
    fmt = BF16 if cfg == 1 else E4M3
    d = ffn = 1024
    for epi, n, k, tail, splits in ((STORE_F32, d, 3 * d, 4, 12), (RESID, d, d, 4, 4), (SWIGLU, 2 * ffn, d, 8, 4),
                                    (RESID, d, ffn, 4, 4)):
        assert library_host().splits(fmt, epi, tokens, n, k) == 1
        assert library_host().workspace_bytes(fmt, epi, tokens, n, k, 1 << 26) == tail * splits * 256 * 256 * 4
    r = np.random.default_rng(tokens)
    cut = np.sort(r.choice(np.arange(1, tokens - 60), 200, replace=False))
    lens = np.diff(np.concatenate([[0], cut, [tokens]]))
    say(f"case: K-split last round, cfg {cfg}, {tokens} tokens in {len(lens)} requests (longest {lens.max()}), 1 step")
    case = make_case(cfg, lens=lens, shape=reduced_shape(d=d, n_q=8, n_kv=2, ffn=ffn, head_hidden=256), n_req=len(lens))
    starts = np.concatenate([[0], cut])
    sample = sorted({0, len(lens) // 2} | set(np.nonzero(starts + lens > 16384)[0].tolist()))
    _against_oracle(case, sample, TOL_HDRAFT[case.fmt], TOL_Z[case.fmt])


@pytest.mark.parametrize("cfg", [1, 4], ids=["bf16", "e4m3"])
@pytest.mark.parametrize("rows", [1, 16, 17, 33, 64])
def test_few_row_gemm_edges(cfg, rows):
    """The few-row kernel: one to four 16-row blocks, full and ragged, K
    ranges that end inside a chunk of activations (ffn 2,688 = 10.5 blocks of
    256), K splits (the d-wide outputs) and the unsplit RoPE and SwiGLU
    epilogues; prompts of one token, so that the prefill has `rows` rows too.
    Tolerance: the repository's bounds for bf16 and e4m3 layers."""
    shape = reduced_shape(d=2048, n_q=16, n_kv=4, ffn=2688, head_hidden=1024)
    say(f"case: few rows, cfg {cfg}, {rows} requests, d=2048, 2 steps")
    case = make_case(cfg, lens=[1] * rows, shape=shape, n_req=rows)
    _against_oracle(case, sorted({0, rows // 2, rows - 1}), TOL_HDRAFT[case.fmt], TOL_Z[case.fmt], steps=2)


@pytest.mark.parametrize("cfg,d", [(1, 1024), (1, 2048), (4, 1024)], ids=["bf16 d=1024", "bf16 d=2048", "e4m3 d=1024"])
@pytest.mark.parametrize("rows", [1, 33])
def test_few_row_gated_qkv(cfg, d, rows):
    """A gated q|k|v narrow enough for the few-row kernel, unsplit: the gate
    columns of its RoPE epilogue.  Tolerance: the repository's bounds for bf16
    and e4m3 layers."""
    fmt, columns = (BF16 if cfg == 1 else E4M3), (2 * 16 + 2 * 4) * 128
    assert library_host().streams(fmt, QKV_ROPE, rows, columns, d)
    assert library_host().splits(fmt, QKV_ROPE, rows, columns, d) == 1
    shape = reduced_shape(d=d, n_q=16, n_kv=4, ffn=1024, head_hidden=256)
    say(f"case: few rows, gated QKV, cfg {cfg}, d={d}, {rows} requests, 2 steps")
    case = make_case(cfg, lens=[1] * rows, shape=shape, n_req=rows, attn_gate=True)
    _against_oracle(case, sorted({0, rows // 2, rows - 1}), TOL_HDRAFT[case.fmt], TOL_Z[case.fmt], steps=2)


@pytest.mark.parametrize("cfg", [1, 4], ids=["bf16", "e4m3"])
@pytest.mark.parametrize("requests", [3, 20, 61])
def test_few_row_results_and_the_rows_beside(cfg, requests):
    """Calls of up to 64 rows on the few-row kernel, in another order of
    requests: the same bits (rows of a call do not meet in any sum).  One
    request alone may take other K splits and page ranges, so it agrees to the
    spread of fp32 summation order (TOL_VARIANT)."""
    shape = reduced_shape(d=2048, n_q=16, n_kv=4, ffn=2688, head_hidden=1024)
    r = np.random.default_rng(requests)
    lens = np.ones(requests, np.int32)
    lens[r.integers(0, requests, min(3, 64 - requests))] += 1
    say(f"case: few rows, cfg {cfg}, {requests} requests ({lens.sum()} rows) permuted and alone")
    case = make_case(cfg, lens=lens, shape=shape, n_req=requests)
    pred = make_predictor(case, max_slots=2 * requests + 1)
    off = np.concatenate([[0], np.cumsum(lens)])
    H, S = device_states(case), device_states(case, step_inputs(case, 1))

    def calls(slots, order):
        rows = np.concatenate([np.arange(off[i], off[i + 1]) for i in order])
        z0, h0 = pred.prefill(slots, lens[order], *[x[rows].contiguous() for x in H], want_hdraft=True)
        z1, h1 = pred.step(slots, *[x[order].contiguous() for x in S], want_hdraft=True)
        z0, h0, z1, h1 = (tensor_to_f64(x) for x in (z0, h0, z1, h1))
        at = np.concatenate([[0], np.cumsum(lens[order])])
        return {i: (z0[k], z1[k], h0[at[k]:at[k + 1]], h1[k]) for k, i in enumerate(order)}

    base = calls(list(range(requests)), list(range(requests)))
    perm = calls(list(range(requests, 2 * requests)), r.permutation(requests).tolist())
    for i in range(requests):
        assert all(np.array_equal(a, b) for a, b in zip(base[i], perm[i])), i
    pred.release(list(range(2 * requests)))
    for i in sorted({0, requests // 2, requests - 1}):
        alone = calls([2 * requests], [i])[i]
        pred.release([2 * requests])
        assert z_errors(np.array(alone[:2]), np.array(base[i][:2])).max() <= TOL_VARIANT, i
        assert rel_fro(alone[2], base[i][2]) <= TOL_VARIANT and rel_fro(alone[3], base[i][3]) <= TOL_VARIANT, i
    pred.close()


@pytest.mark.parametrize("cfg", [1, 4], ids=["bf16", "e4m3"])
@pytest.mark.parametrize("rows", [1, 33])
def test_few_row_gemm_too_wide_for_one_round(cfg, rows):
    """A gated q|k|v of more rows than the few-row kernel's workgroups cover in
    one round (10,240 bf16, 18,432 e4m3): K splits of the tiles and their
    RoPE reduce.  Tolerance: the repository's bounds for bf16 and e4m3."""
    shape = reduced_shape(d=1024, n_q=64 if cfg == 4 else 32, n_kv=8, ffn=1024)
    say(f"case: few rows, wide gated QKV, cfg {cfg}, {rows} requests, 1 step")
    case = make_case(cfg, lens=[1] * rows, shape=shape, n_req=rows, attn_gate=True)
    _against_oracle(case, sorted({0, rows // 2, rows - 1}), TOL_HDRAFT[case.fmt], TOL_Z[case.fmt])


@pytest.mark.parametrize("cfg,lens", [
    (1, [1, 15, 16, 17, 500, 1007]),            # one workgroup per request: up to 64 pages, waves without pages
    (1, [1007, 1023, 30]),                      # the step crosses 64 pages in one request: ranges instead
    (4, [3, 64, 129, 250] * 3),                 # 8 query heads per KV head
    (1, [5] * 150 + [110] * 20),                # 8 pages at most, hundreds of workgroups
    (1, [4100, 40, 2000]),                      # more than 8 records per request: four merge groups
], ids=["short", "at 64 pages", "gqa8", "many short", "many records"])
def test_decode_attention_by_request_and_by_ranges(cfg, lens):
    """Steps around the rule that picks one workgroup per request or page
    ranges, and around the merge's record groups.  Tolerance: the
    repository's bounds for bf16 and e4m3 layers."""
    n_q, n_kv = (16, 2) if cfg == 4 else (8, 2)
    say(f"case: decode attention, cfg {cfg}, {len(lens)} requests of up to {max(lens)} tokens, 2 steps")
    case = make_case(cfg, lens=lens, shape=reduced_shape(n_q=n_q, n_kv=n_kv), n_req=len(lens))
    sample = sorted({0, len(lens) // 2, len(lens) - 1, int(np.argmax(lens))})
    _against_oracle(case, sample, TOL_HDRAFT[case.fmt], TOL_Z[case.fmt], steps=2)


@pytest.mark.parametrize("lens", [[1], [33, 31, 64, 7], [40] * 129], ids=["1 tile", "ragged tiles", "258 tiles"])
def test_final_norm_pooling_row_groups(lens):
    """Pooling tiles of one row, of ragged row groups, and past the switch to
    one group per tile (256 tiles).  Tolerance: the bf16 layer's bounds."""
    say(f"case: pooling tiles, {len(lens)} requests of up to {max(lens)} tokens")
    case = make_case(1, lens=lens, shape=reduced_shape(d=1024, n_q=8, n_kv=2, ffn=1024), n_req=len(lens))
    _against_oracle(case, sorted({0, len(lens) // 2, len(lens) - 1}), TOL_HDRAFT["bf16"], TOL_Z["bf16"])


@pytest.mark.parametrize("cfg,shape", [(0, dict(d=256, n_q=4, n_kv=2, ffn=256, head_hidden=128)),
                                       (1, dict(d=2048, n_q=16, n_kv=4, ffn=2688, head_hidden=256))],
                         ids=["norm", "summing norm"])
@pytest.mark.parametrize("lens", [[1], [63, 64, 65], [300, 1, 16, 17, 2], [3] * 257], ids=["1", "3", "5", "257"])
def test_metadata_beside_the_first_norm(cfg, shape, lens):
    """The metadata block fetched by extra blocks of the first norm: one wave
    per request (request counts around four and past a block of waves, tokens
    around a wave), in the prefill and in two steps.  Whole numbers, exact."""
    from paper_2609_01068_amd import binding as B
    say(f"case: metadata, cfg {cfg}, {len(lens)} requests of up to {max(lens)} tokens, 2 steps")
    case = make_case(cfg, lens=lens, shape=reduced_shape(**shape), n_req=len(lens))
    n, slots = len(lens), list(range(len(lens)))[::-1]
    pred = make_predictor(case, max_seq_len=max(lens) + 32)

    def check(pos, lens):
        assert np.array_equal(pred.meta(B.OUTLETS_META_DEV_POSITIONS), pos)
        assert np.array_equal(pred.meta(B.OUTLETS_META_DEV_CU_SEQLENS), np.concatenate([[0], np.cumsum(lens)]))
        assert np.array_equal(pred.meta(B.OUTLETS_META_DEV_LAST_IDX), np.cumsum(lens) - 1)
        assert np.array_equal(pred.meta(B.OUTLETS_META_DEV_TOKEN_SLOT), np.repeat(slots, lens))
        table = pred.meta(B.OUTLETS_META_PAGE_TABLE)
        assert np.array_equal(pred.meta(B.OUTLETS_META_DEV_PAGE_TABLE)[table >= 0], table[table >= 0])

    pred.prefill(slots, case.lens, *device_states(case))
    check(np.concatenate([np.arange(x) for x in lens]), lens)
    for k in (1, 2):
        pred.step(slots, *device_states(case, step_inputs(case, k)))
        check(np.asarray(lens) + k - 1, [1] * n)
    pred.close()


@pytest.mark.parametrize("cfg,shape", [(0, dict(d=256, n_q=4, n_kv=2, ffn=256, head_hidden=128)),
                                       (1, dict(d=2048, n_q=16, n_kv=4, ffn=2688, head_hidden=256))],
                         ids=["fp32", "bf16"])
@pytest.mark.parametrize("groups", [["META"], None], ids=["only metadata", "all groups"])
def test_metadata_group_is_timed(cfg, shape, groups):
    """Each call records one launch of the metadata group while it is timed,
    and gives the same results, bit for bit, as without timing."""
    lens = [33, 1, 16, 64, 17]
    say(f"case: metadata timing, cfg {cfg}, groups {groups}, {len(lens)} requests, 3 steps")
    case = make_case(cfg, lens=lens, shape=reduced_shape(**shape), n_req=len(lens))
    slots = list(range(len(lens)))
    runs = []
    for timed in (False, True):
        pred = make_predictor(case)
        if timed:
            pred.profile(True, groups=groups)
        out = list(pred.prefill(slots, case.lens, *device_states(case), want_hdraft=True))
        for k in (1, 2, 3):
            out += pred.step(slots, *device_states(case, step_inputs(case, k)), want_hdraft=True)
        runs.append([tensor_to_f64(x) for x in out])
        if timed:
            for call, n in (("prefill", 1), ("step", 3)):
                ms, launches = pred.profile_read(call)["META"]
                assert launches == n and ms > 0.0, call
        pred.close()
    for a, b in zip(*runs):
        assert np.array_equal(a, b)
