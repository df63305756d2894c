"""What calls launch, seen from the host (tests/launches.py): which kernels serve which shapes, and that a call that fails has
launched nothing.  No GPU is touched."""
import pytest

import test_gpu_attn_one_block as one_block
import test_gpu_score_packed as packed
import test_gpu_score_sweeps as sweeps
from launches import AT, launches


def score(hq, hkv, d, n_text, n_video, layers=None, **more):
    n_keys = n_video + n_text
    args = dict(q_text=AT, q_tok_stride=hq * d, q_head_stride=d, k_cache=AT, k_tok_stride=hkv * d, k_head_stride=d, batch=1,
                n_text=n_text, n_keys=n_keys, n_video=n_video, text_pos0=-1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                softmax_scale=0.125, scores=AT, workspace=AT, workspace_bytes=1 << 40)
    if layers:
        args.update(n_layers=layers, q_layer_stride=n_text * hq * d, k_layer_stride=n_keys * hkv * d)
    args.update(more)
    return ("specvlm_score_layers" if layers else "specvlm_score", args)


def attn(hq, hkv, d, q_len, kv_len, **more):
    args = dict(q=AT, q_tok_stride=hq * d, q_head_stride=d, k=AT, v=AT, kv_tok_stride=hkv * d, kv_head_stride=d, batch=1, q_len=q_len,
                kv_len=kv_len, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, softmax_scale=0.125, out=AT, workspace=AT,
                workspace_bytes=1 << 40)
    args.update(more)
    return ("specvlm_decode_attn", args)


# each with so much LDS that the kernel's attribute has to be raised first
@pytest.mark.parametrize("call", [score(8, 4, 64, 64, 1568), score(8, 1, 128, 64, 700, row_lse=AT), attn(14, 2, 64, 1, 1511),
                                  attn(64, 8, 128, 6, 12806), attn(64, 8, 128, 1, 1000)])
def test_a_call_that_fails_has_launched_nothing(call, tmp_path):
    no_device, no_attribute, good = launches([(*call, 1, 0), (*call, 0, 1), call], tmp_path)
    assert no_device == (-4, []) and no_attribute == (-4, [])
    assert good[0] == 0 and len(good[1]) >= 1


def accept(batch, gamma, vocab, **more):
    return ("specvlm_accept", dict(target_logits=AT, draft_logits=AT, draft_tokens=AT, uniforms=AT, batch=batch, gamma=gamma, vocab=vocab,
                                   temperature=1, n_accepted=AT, out_tokens=AT, workspace=AT, workspace_bytes=1 << 40, **more))


# workgroups of the second sampling pass: as many as CUs are the last that count themselves in
@pytest.mark.parametrize("batch,vocab,one", [(1, 152064, True), (13, 152064, True), (14, 152064, False), (256, 8192, True), (257, 8192, False),
                                             (128, 8193, True), (129, 8193, False), (5000, 1024, True)])
def test_sampling_counts_arrivals_only_up_to_one_workgroup_per_cu(batch, vocab, one, tmp_path):
    [(status, got)] = launches([accept(batch, 2, vocab)], tmp_path)
    chunk = 1024 if vocab <= 1024 else 8192
    chunks = -(-vocab // chunk)
    assert status == 0
    assert [(name, grid) for name, grid, _, _ in got] == [(f"accept_softmax_partial<{chunk}>", (chunks, 5, batch))] + (
        [(f"accept_sample_kernel<{chunk}, 0>", (chunks, batch, 1))] if one else
        [(f"accept_sample_kernel<{chunk}, 1>", (chunks, batch, 1)), (f"accept_sample_kernel<{chunk}, 2>", (1, batch, 1))])


def least_bytes(batch, gamma, vocab):
    """What sampling needs: two statistics a row and chunk, two numbers a row, one a chunk, one a request (each 256-byte aligned)."""
    rows, chunks = 2 * gamma + 1, -(-vocab // 8192)
    return sum((n * 4 + 255) // 256 * 256 for n in (batch * rows * chunks, batch * rows * chunks, batch * rows * 2, batch * chunks, batch))


# (the query asks for the segments' masses as well: 16 numbers a chunk, without which the call is slower)
@pytest.mark.parametrize("batch,gamma,vocab", [(1, 7, 152064), (20, 3, 152064), (3, 0, 1000), (2, 64, 8193)])
def test_sampling_does_without_the_segments_masses(batch, gamma, vocab, tmp_path):
    least = least_bytes(batch, gamma, vocab)
    query = ("specvlm_accept_workspace_bytes", dict(batch=batch, gamma=gamma, vocab=vocab, sampling=1))
    calls = [accept(batch, gamma, vocab) for _ in range(3)]
    for (_, args), n in zip(calls, (1 << 40, least, least - 1)):
        args["workspace_bytes"] = n
    (asked, _), full, enough, short = launches([query, *calls], tmp_path)
    assert asked == least + (batch * -(-vocab // 8192) * 64 + 255) // 256 * 256
    assert full[0] == 0 and enough == full and short == (-3, [])


@pytest.mark.parametrize("batch,n,tokens,pair", [(1, 12544, 16, False), (256, 4096, 4, False), (257, 4096, 4, True), (257, 4097, 16, True),
                                                 (257, 16385, 32, True), (1000, 32769, 64, False)])
def test_selections_share_a_cu_where_the_requests_are_more_than_the_cus(batch, n, tokens, pair, tmp_path):
    args = dict(scores=AT, cu_video=AT, k_top=AT, keep_budget=AT, cu_keep=AT, batch=batch, max_n_video=n, total_keep=batch, keep_idx=AT)
    [(status, got)] = launches([("specvlm_select", args)], tmp_path)
    assert status == 0 and [l[:3] for l in got] == [(f"select_kernel<{tokens}, {'true' if pair else 'false'}>", (batch, 1, 1), (1024, 1, 1))]


def test_the_sweeps_shapes_take_the_sweeps(tmp_path):
    def call(layers, V, L, P, hq, hkv, d, mode, text_pos0=None):
        more = dict(n_keys=P + V + L, video_start=P, norm_mode=mode, text_pos0=P + V if text_pos0 is None else text_pos0)
        return score(hq, hkv, d, L, V, layers, **more)

    got = launches([call(2, *shape) for shape, _ in sweeps.KEY_SPLITS], tmp_path)
    for (shape, splits), (status, ls) in zip(sweeps.KEY_SPLITS, got):
        d, grid = shape[5], (2 * splits + 7) // 8 * 8                 # two layers, a multiple of the XCDs
        assert status == 0 and [l[0] for l in ls[:3]] == [f"score_sweep_kernel<{d}, 0>", f"score_lse_kernel<{1 if splits <= 8 else 8}>",
                                                          f"score_sweep_kernel<{d}, 1>"], (shape, ls)
        assert ls[0][1] == (grid, 1, 1), (shape, ls)
    got = launches([call(*shape) for shape, _ in sweeps.PARTIAL_COLUMNS], tmp_path)
    for (shape, columns), (status, ls) in zip(sweeps.PARTIAL_COLUMNS, got):
        blocks = (shape[1] + 255) // 256
        assert status == 0 and ls[2][1] == ((blocks * columns + 7) // 8 * 8, 1, 1), (shape, ls)
        assert ls[3][0] == f"score_final_kernel<{'1, 8' if columns <= 8 else '1, 16' if columns <= 16 else '8, 16'}>", (shape, ls)
    got = launches([call(None, V, L, 0, hq, hkv, d, mode, pos0) for V, L, pos0, hq, hkv, d in sweeps.INSIDE for mode in (0, 1)] +
                   [call(None, 2200, 70, 0, 10, 2, 64, 0)], tmp_path)
    assert all(status == 0 and [l[0].split("<")[0] for l in ls] == ["score_sweep_kernel", "score_lse_kernel", "score_sweep_kernel",
                                                                    "score_final_kernel"] for status, ls in got)


@pytest.mark.parametrize("hq,hkv,d,L,V,lse,small", [(4, 1, 64, 64, 1568, False, True), (8, 1, 64, 64, 17344, False, True), (8, 1, 64, 64, 17345, False, False),
                                                    (9, 1, 64, 64, 500, False, False), (4, 4, 64, 65, 700, False, True), (8, 1, 128, 64, 300, True, True),
                                                    (8, 2, 128, 64, 300, False, False), (1, 1, 64, 513, 300, True, False)])
def test_one_small_layer_takes_the_two_launch_form(hq, hkv, d, L, V, lse, small, tmp_path):
    [(status, ls)] = launches([score(hq, hkv, d, L, V, row_lse=AT if lse else None)], tmp_path)
    assert status == 0
    if small:
        assert [l[0] for l in ls] == [f"score_small_rows_kernel<{d}>"] * (not lse) + [f"score_small_cols_kernel<{d}>"]
    else:
        assert ls[-2][0] == f"score_sweep_kernel<{d}, 1>"


def test_the_packed_shapes_have_fewer_rows_in_the_workspace_of_before(tmp_path):
    def call(layers, V, L, P, hq, hkv, d, mode):
        return score(hq, hkv, d, L, V, layers, n_keys=P + V + L, video_start=P, norm_mode=mode, text_pos0=P + V)

    shapes = [(s, n) for s, n in packed.PACKED] + [((1, V, L, 0, hq, hkv, d, 0), 1) for V, L, _, hq, hkv, d in packed.INSIDE]
    for (shape, blocks), (status, ls) in zip(shapes, launches([call(*s) for s, _ in shapes], tmp_path, words=True)):
        assert padded(ls[2], shape[2], shape[1], sum(shape[1:4]), shape[3]) == (shape[2] + 15) // 16 * 16, (shape, ls)
        assert status == 0 and ls[0][0] == f"score_sweep_kernel<{shape[6]}, 0>", (shape, ls)
        rows_a_block = 256 if ls[1][0] == "score_lse_kernel<1>" else 32
        assert ls[1][1] == (blocks * 256 // rows_a_block, shape[5], shape[0]), (shape, ls)
    # what the call asks for is what 64 rows a tile took: a layer's (max, sum) pairs, normalisers and columns, by the splits it had
    layers, V, L, hq, hkv, d = 24, 12544, 85, 64, 8, 128
    query = ("specvlm_score_layers_workspace_bytes", dict(n_layers=layers, batch=1, n_text=L, n_keys=V + L, n_video=V, n_q_heads=hq, n_kv_heads=hkv,
                                                          head_dim=d))
    least = layers * hkv * 4 * (1024 * 2 + 1024 + 12544)
    (asked, _), enough, short = launches([query, score(hq, hkv, d, L, V, layers, workspace_bytes=least),
                                          score(hq, hkv, d, L, V, layers, workspace_bytes=least - 1)], tmp_path)
    assert asked == least and enough[0] == 0 and short == (-3, [])


# (a q head's queries as the sweeps pad them: the word of their parameters that comes nine behind n_text, n_keys, video_start and n_video)
def padded(launch, n_text, n_video, n_keys, video_start=0):
    words = launch[4]
    at = [i for i in range(20) if words[i:i + 4] == [n_text, n_keys, video_start, n_video]]
    assert len(at) == 1, words
    return words[at[0] + 9]


@pytest.mark.parametrize("hq,hkv,d,n_text,n_video,layers,pad", [
    (32, 32, 128, 13, 12544, None, 64), (32, 32, 128, 28, 3000, 24, 64), (16, 16, 64, 9, 3000, 24, 64), (16, 16, 64, 32, 12544, None, 64),
    (16, 8, 128, 13, 12544, None, 16), (64, 8, 128, 28, 3000, 24, 32), (6, 3, 64, 32, 3000, 24, 32), (16, 16, 64, 130, 700, 24, 192)])
def test_queries_are_packed_only_where_the_sweeps_have_less_to_do(hq, hkv, d, n_text, n_video, layers, pad, tmp_path):
    [(status, ls)] = launches([score(hq, hkv, d, n_text, n_video, layers)], tmp_path, words=True)
    assert status == 0 and [l[0] for l in ls[::2]][:2] == [f"score_sweep_kernel<{d}, 0>", f"score_sweep_kernel<{d}, 1>"]
    assert padded(ls[0], n_text, n_video, n_text + n_video) == padded(ls[2], n_text, n_video, n_text + n_video) == pad


# (given normalisers: pass B alone)
@pytest.mark.parametrize("hq,hkv,d,n_text,n_video,layers,pad", [
    (7, 1, 128, 104, 8343, 24, 128), (14, 2, 64, 327, 17529, 2, 384), (40, 8, 128, 303, 9187, None, 320), (4, 1, 64, 458, 16508, 24, 512),
    (64, 8, 128, 85, 12544, 24, 96), (28, 4, 128, 200, 25088, 28, 208), (4, 1, 64, 263, 28130, 8, 272)])
def test_with_given_normalisers_queries_are_packed_for_more(hq, hkv, d, n_text, n_video, layers, pad, tmp_path):
    [(status, ls)] = launches([score(hq, hkv, d, n_text, n_video, layers, row_lse=AT)], tmp_path, words=True)
    assert status == 0 and ls[1][0] == f"score_sweep_kernel<{d}, 1>"
    assert padded(ls[1], n_text, n_video, n_text + n_video) == pad


# one block of query rows: roles only where the cache is streamed (8 MB), the splits are of 128 keys and more and the workgroups of head size 64
# fit one round of one to a CU or take several
@pytest.mark.parametrize("hq,hkv,d,batch,kv_len,splits,loaders", [
    (7, 1, 128, 1, 16383, 64, False), (7, 1, 128, 1, 16384, 64, True), (28, 4, 128, 1, 4161, 33, False), (14, 2, 64, 1, 16383, 32, False),
    (14, 2, 64, 1, 16384, 32, True), (14, 2, 64, 1, 32768, 128, True), (14, 2, 64, 1, 33024, 129, False), (16, 8, 64, 1, 16384, 64, False),
    (16, 8, 64, 1, 16640, 65, True), (16, 8, 64, 65, 128, 0, True), (8, 4, 64, 65, 1500, 0, False), (8, 4, 64, 100, 600, 0, False),
    (64, 8, 128, 1, 16384, 64, False), (64, 8, 128, 1, 16128, 63, True), (64, 8, 128, 1, 16448, 64, True), (28, 4, 128, 1, 32768, 128, True),
    (64, 8, 128, 65, 256, 0, False), (64, 8, 128, 65, 257, 0, True), (64, 8, 128, 8, 255, 0, False), (64, 8, 128, 8, 256, 0, True),
    (40, 8, 128, 8, 1100, 0, True), (28, 4, 128, 2, 1100, 0, False), (14, 2, 64, 8, 9000, 0, False),
    (7, 1, 128, 1, 2097, 3, False), (7, 1, 128, 1, 2098, 3, True), (12, 3, 128, 1, 1399, 2, True), (4, 1, 64, 1, 30000, 8, False),
    *((2 * hkv, hkv, d, 1, 164 * splits, splits, True) for d, hkv, splits in one_block.STREAMED)])
def test_one_row_block_has_loader_waves_where_memory_is_what_it_waits_for(hq, hkv, d, batch, kv_len, splits, loaders, tmp_path):
    more = dict(batch=batch, cu_q=AT, cu_kv=AT) if batch > 1 else {}
    [(status, got)] = launches([attn(hq, hkv, d, 1, kv_len, num_splits=splits, **more)], tmp_path)
    assert status == 0
    assert got[0][0].startswith(f"attn_split_kernel<{d}, 1, " + ("2, 64, " if loaders else "4, 128, 2, 0, ")), got


# head size 64: four stages where a workgroup has a CU to itself, in one round that is not full or with splits of 640 keys, and in several rounds of those
@pytest.mark.parametrize("hq,hkv,batch,q_len,kv_len,splits,stages", [
    (14, 2, 1, 1, 30000, 0, 4), (14, 2, 1, 4, 30000, 0, 4), (14, 2, 1, 8, 3000, 0, 4), (10, 5, 1, 4, 100000, 0, 4), (14, 2, 1, 6, 30600, 102, 4),
    (14, 2, 1, 6, 30900, 103, 3), (14, 2, 1, 6, 65792, 103, 3), (14, 2, 1, 6, 65920, 103, 4), (14, 2, 1, 26, 12000, 0, 3), (14, 2, 1, 26, 30000, 0, 4),
    (16, 8, 1, 20, 30000, 0, 3), (16, 8, 1, 50, 30000, 0, 4), (14, 2, 1, 6, 100000, 129, 3), (14, 2, 65, 6, 1500, 0, 3), (8, 4, 128, 8, 3000, 0, 4),
    (8, 4, 8, 24, 20480, 32, 4), (8, 4, 8, 24, 20448, 32, 3), (14, 2, 5, 6, 20000, 0, 3)])
def test_the_ring_of_head_size_64(hq, hkv, batch, q_len, kv_len, splits, stages, tmp_path):
    more = dict(batch=batch, cu_q=AT, cu_kv=AT) if batch > 1 else {}
    [(status, got)] = launches([attn(hq, hkv, 64, q_len, kv_len, num_splits=splits, **more)], tmp_path)
    assert status == 0
    shape = [int(x) for x in got[0][0].split("<")[1].split(",")[:6]]
    assert shape[0] == 64 and shape[2:5] == [2, 64, stages], got


@pytest.mark.parametrize("hq,hkv,q_len,kv_len,splits", [(16, 8, 1, 30000, 0), (16, 8, 20, 30000, 0), (16, 16, 4, 50000, 6), (16, 8, 1, 8400, 3)])
def test_the_ring_of_eight_heads_of_size_64_is_deep_where_a_heads_keys_lie_together(hq, hkv, q_len, kv_len, splits, tmp_path):
    apart = dict(kv_tok_stride=64, kv_head_stride=64 * kv_len)
    both = launches([attn(hq, hkv, 64, q_len, kv_len, num_splits=splits, **more) for more in ({}, apart)], tmp_path)
    assert [got[0][0].split(",")[4].strip() for _, got in both] == ["3", "4"], both


@pytest.mark.parametrize("hq,hkv,d,batch,q_len,splits,kernel", [
    (64, 8, 128, 8, 1, 64, "8, 384, false"), (64, 8, 128, 9, 1, 64, "4, 384, true"), (64, 8, 128, 8, 8, 36, "3, 384, false"),
    (64, 8, 128, 8, 8, 37, "4, 384, true"), (14, 2, 64, 8, 4, 200, "22, 192, false"), (14, 2, 64, 8, 8, 200, "4, 192, true"),
    (32, 4, 64, 4, 4, 40, "4, 192, false"), (32, 4, 128, 5, 4, 100, "4, 384, true"), (4, 1, 64, 8, 2, 100, "16, 192, false")])
def test_the_merge_of_many_rows_goes_in_rounds(hq, hkv, d, batch, q_len, splits, kernel, tmp_path):
    [(status, got)] = launches([attn(hq, hkv, d, q_len, 128 * splits, num_splits=splits, batch=batch, cu_q=AT, cu_kv=AT)], tmp_path)
    assert status == 0 and got[1][0] == f"attn_merge_kernel<{d}, {kernel}>" and got[1][1] == (hq * q_len * batch, 1, 1), got
