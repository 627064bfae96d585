"""GPU parity of harli_decode_step against the CPU oracle (through the C ABI).

Bar: page-table / block indexing bit-exact (the set of slab elements the step changes is
exactly the oracle's); fp outputs max-abs error <= 2e-2 * max|ref| and relative Frobenius
error <= 5e-3 for bf16 storage with fp32 accumulation.
"""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as wl
from paper_2511_11729_amd import binding as hb
from tests.gpu_util import DEV, DecodeCase, assert_close

pytestmark = pytest.mark.gpu


def variant(idx, **kw):
    w = wl.workload(idx)
    return w, dataclasses.replace(w.model, **kw)


# fp32 storage and arithmetic: unit round-off 6e-8, dot products of up to ~700 terms summed lane-wise then by a
# butterfly (error ~ sqrt(K) u), seven chained steps and an fp32 exp -- 1e-4 of the largest output and 2e-5 in
# relative Frobenius norm leave a factor ~10 of slack.
F32_BAR = dict(max_ratio=1e-4, fro=2e-5)


def run_case(w, m, lengths, **kw):
    case = DecodeCase(w, m, np.asarray(lengths, np.int32), **kw)
    y = case.run_gpu()
    ref = case.run_oracle()
    bar = F32_BAR if m.dtype == "f32" else {}
    stats = assert_close(y, ref, "decode output", **bar)
    n = case.check_cache(*((1e-4, 2e-5) if m.dtype == "f32" else ()))
    assert n == len(lengths) * m.n_layers * 2 * m.n_kv * m.head_dim
    return case, stats


def test_tiny_bf16_config0_shapes():
    """Config 0's shapes (hidden 256, 4 x 64 heads, ffn 688 = 43 tiles, ragged) stored as bf16."""
    w, m = variant(0, dtype="bf16")
    run_case(w, m, wl.draw_lengths(w), block_bytes=64 << 10)


@pytest.mark.parametrize("lengths", [
    [0], [0, 1, 15, 16, 17], [255, 256, 257, 511, 512], [700, 3, 1300], [31] * 16, [40] * 17, list(range(5, 105, 3)),
])
def test_tiny_edge_lengths_and_batches(lengths):
    """Empty cache, page boundaries (15/16/17), chunk boundaries (255/256/257), ragged mixes,
    batch 16/17 (one and two MFMA column tiles) and 34 (three)."""
    w, m = variant(0, dtype="bf16")
    run_case(w, m, lengths, block_bytes=64 << 10)


def test_batch_above_64_runs_in_passes():
    w, m = variant(0, dtype="bf16")
    run_case(w, m, [7 + (i * 5) % 90 for i in range(100)], block_bytes=64 << 10)


def test_three_layers_at_batch_250_with_embedding_and_logits():
    """Above 32 sequences the layer GEMMs take the tiled path: here one batch tile of 256 rows with 250 real ones (the
    last 16-row group ragged), a ragged last weight tile (ffn 688 of 768), three layers chained through the row norms
    and the output layer after them."""
    w, m = variant(0, dtype="bf16", n_layers=3, vocab=1000)
    lengths = np.asarray([(i * 29) % 150 for i in range(250)], np.int32)
    case = DecodeCase(w, m, lengths, full_model=True, block_bytes=64 << 10)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (250,))
    hid = case.run_gpu(token_ids=tok)
    ref_hid, ref_logits, _ = case.run_oracle(token_ids=tok)
    assert_close(hid, ref_hid, "hidden state")
    assert_close(case.logits_dev.cpu().numpy(), ref_logits, "logits")
    case.check_cache()
    first = (case.y_dev.clone(), case.logits_dev.clone(), case.slab.clone())
    case.slab.copy_(torch.from_numpy(case.img0.view(np.uint8)))
    case.run_gpu(token_ids=tok)                      # the partial tiles are added in a fixed order: the same bits again
    assert torch.equal(case.y_dev, first[0]) and torch.equal(case.logits_dev, first[1]) and torch.equal(case.slab, first[2])


def test_a_context_for_large_batches_serves_small_ones_on_the_streaming_kernels():
    """max_batch decides whether the workspace of the tiled path exists; the batch of the step decides the path: a step
    of 9 sequences gives the same bits in a context made for 200 as in one made for 9."""
    w, m = variant(0, dtype="bf16", n_layers=2)
    lengths = np.asarray([12, 200, 0, 77, 300, 33, 5, 129, 64], np.int32)
    small = DecodeCase(w, m, lengths, block_bytes=64 << 10)
    roomy = DecodeCase(w, m, lengths, block_bytes=64 << 10, max_batch=200)
    assert roomy.ctx.device_bytes().decode_workspace > small.ctx.device_bytes().decode_workspace
    assert np.array_equal(np.asarray(small.run_gpu()), np.asarray(roomy.run_gpu()))


def test_out_of_range_page_id_is_reported_at_large_batch():
    from paper_2511_11729_amd import binding as hb
    w, m = variant(0, dtype="bf16")
    case = DecodeCase(w, m, np.asarray([20 + i % 30 for i in range(80)], np.int32), block_bytes=64 << 10)
    case.table_dev[70, 1] = 10_000_000
    with pytest.raises(hb.HarliError) as e:
        case.run_gpu()
    assert "page id" in str(e.value)
    case.table_dev[70, 1] = int(case.table[70, 1])
    case.run_gpu()


@pytest.mark.parametrize("n_q,n_kv,d", [(8, 2, 64), (8, 8, 128), (8, 4, 128), (8, 2, 128), (8, 1, 128), (6, 2, 128), (5, 1, 128),
                                        (6, 1, 128), (7, 1, 128)])
def test_head_layouts(n_q, n_kv, d):
    """GQA ratios 1, 2, 4, 8 and both head sizes."""
    w, m = variant(0, dtype="bf16", hidden=n_q * d // 2, n_q=n_q, n_kv=n_kv, head_dim=d, ffn=320)
    run_case(w, m, [0, 37, 300, 16], block_bytes=256 << 10)


@pytest.mark.parametrize("G", [5, 6, 7, 8])
def test_matrix_unit_attention_at_the_edges_of_pages_and_chunks(G):
    """Groups of five to eight query heads: the last token at the end and at the start of a page, of a wave's 32 tokens and
    of a chunk of 128; two KV heads."""
    w, m = variant(0, dtype="bf16", hidden=G * 128, n_q=2 * G, n_kv=2, head_dim=128, ffn=320)
    run_case(w, m, [15, 31, 32, 126, 127, 128, 255, 256], block_bytes=256 << 10)


def test_non_dividing_page_size():
    """Pages that do not divide the block (3 per 64 KiB block with slack), several chunks."""
    w, m = variant(0, dtype="bf16", hidden=640, n_q=5, n_kv=5, head_dim=128, ffn=256)
    case, _ = run_case(w, m, [100, 33, 250], block_bytes=64 << 10)
    assert case.geom.pages_per_block == 3 and case.pool.stats().kv_chunks > 3


def test_three_layer_model_with_embedding_and_logits():
    w, m = variant(0, dtype="bf16", n_layers=3, vocab=1000)
    lengths = [12, 200, 0, 77]
    case = DecodeCase(w, m, np.asarray(lengths, np.int32), full_model=True, block_bytes=64 << 10)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (4,))
    hid = case.run_gpu(token_ids=tok)
    ref_hid, ref_logits, ref_next = case.run_oracle(token_ids=tok)
    assert_close(hid, ref_hid, "hidden state")
    logits = case.logits_dev.cpu().numpy()
    assert_close(logits, ref_logits, "logits")
    case.check_cache()
    nxt = case.next_dev.cpu().numpy()
    # argmax is exact on the GPU's own logits (ties to the lowest index) ...
    assert np.array_equal(nxt, np.argmax(logits, axis=-1))
    # ... and equals the oracle's wherever the oracle's top-2 gap exceeds the tolerance
    srt = np.sort(ref_logits, axis=-1)
    clear = (srt[:, -1] - srt[:, -2]) > 4e-2 * np.max(np.abs(ref_logits))
    assert np.array_equal(nxt[clear], ref_next[clear])


def test_step_is_bit_reproducible():
    """The same step gives the same bits every time, on any stream and whatever ran in between (the row norms are
    summed across workgroups as integers, in which the order of arrival does not matter)."""
    w, m = variant(0, dtype="bf16", n_layers=3, vocab=1000)
    lengths = [12, 200, 0, 77, 300, 33, 5, 129, 64]
    case = DecodeCase(w, m, np.asarray(lengths, np.int32), full_model=True, block_bytes=64 << 10)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (len(lengths),))
    case.run_gpu(token_ids=tok)
    first = (case.y_dev.clone(), case.logits_dev.clone(), case.next_dev.clone(), case.slab.clone())
    side = torch.cuda.Stream()
    busy = torch.randn(2048, 2048, device="cuda:0")
    for rep in range(6):
        case.slab.copy_(torch.from_numpy(case.img0.view(np.uint8)))
        if rep % 2:                                   # unrelated work on another stream while the step runs
            with torch.cuda.stream(side):
                for _ in range(4):
                    busy = busy @ busy * 1e-3
        case.run_gpu(token_ids=tok, stream=side if rep >= 3 else None)
        assert torch.equal(case.y_dev, first[0]) and torch.equal(case.logits_dev, first[1])
        assert torch.equal(case.next_dev, first[2]) and torch.equal(case.slab, first[3])


def test_argmax_ties_go_to_the_lowest_index():
    w, m = variant(0, dtype="bf16", n_layers=1, vocab=64)
    def same_rows(case):             # identical rows in the output layer give exactly equal logits
        case.extras_np["wlm"][5] = case.extras_np["wlm"][40]
    case = DecodeCase(w, m, np.asarray([3, 9], np.int32), full_model=True, block_bytes=64 << 10, tweak=same_rows)
    case.run_gpu(token_ids=[1, 2])
    logits = case.logits_dev.cpu().numpy()
    assert np.array_equal(logits[:, 5], logits[:, 40])
    assert np.array_equal(case.next_dev.cpu().numpy(), np.argmax(logits, axis=-1))


def test_out_of_range_page_id_is_reported_not_dereferenced():
    from paper_2511_11729_amd import binding as hb
    w, m = variant(0, dtype="bf16")
    case = DecodeCase(w, m, np.asarray([20, 40], np.int32), block_bytes=64 << 10)
    case.table_dev[1, 1] = 10_000_000
    with pytest.raises(hb.HarliError) as e:
        case.run_gpu()
    assert "page id" in str(e.value)
    case.table_dev[1, 1] = int(case.table[1, 1])
    case.run_gpu()                                   # the flag was cleared; a clean step passes


def test_config1_full_size_layer():
    """The 7B-class layer at its real shape: batch 8, lengths uniform in [256, 2048]."""
    w = wl.workload(1)
    case, stats = run_case(w, w.model, wl.draw_lengths(w))
    print("config 1 decode parity: max-abs ratio %.2e, rel-Fro %.2e" % stats)


def test_two_steps_in_a_row_use_the_appended_token():
    """Step t+1 attends to the K/V that step t appended (same context, same pages)."""
    w, m = variant(0, dtype="bf16")
    lengths = np.asarray([14, 30, 250], np.int32)
    case = DecodeCase(w, m, lengths, block_bytes=64 << 10)
    y1 = case.run_gpu()
    ref1 = case.run_oracle()
    assert_close(y1, ref1, "step 1")
    # second step: feed y1 back in as the next input on both sides
    case.x_dev.copy_(torch.from_numpy(ref1.astype(np.float32)))
    case.kv_len_dev += 1
    case.ctx.decode_step(batch=3, kv_len=case.kv_len_dev, page_table=case.table_dev, max_pages=case.max_pages,
                         max_kv_len=int(lengths.max()) + 2, x_in=case.x_dev, x_out=case.y_dev)
    torch.cuda.synchronize()
    case.ctx.check()
    from oracle import harli_oracle as O
    from tests.gpu_util import shapes_of
    ref2 = O.decode_model_paged(ref1.astype(np.float32), case.layers_np, None, shapes_of(m), case.okv, lengths + 1, case.table)
    assert_close(case.y_dev.cpu().numpy(), ref2, "step 2")


# ---- fp32 storage (config 0 as written): every tensor fp32, generic kernels without tile restrictions ----

def test_config0_fp32_as_written():
    w = wl.workload(0)
    assert w.model.dtype == "f32"
    case, stats = run_case(w, w.model, wl.draw_lengths(w), block_bytes=64 << 10)
    print("config 0 fp32 decode parity: max-abs ratio %.2e, rel-Fro %.2e" % stats)


@pytest.mark.parametrize("lengths", [[0], [0, 1, 15, 16, 17], [255, 256, 257], [31] * 17, list(range(5, 105, 9))])
def test_fp32_edge_lengths_and_batches(lengths):
    """Empty cache, page boundaries, a batch that spans three 8-row tiles."""
    w = wl.workload(0)
    run_case(w, w.model, lengths, block_bytes=128 << 10)


@pytest.mark.parametrize("hidden,n_q,n_kv,d,ffn", [(200, 6, 2, 20, 333), (96, 3, 1, 34, 70), (320, 2, 2, 160, 64)])
def test_fp32_arbitrary_shapes(hidden, n_q, n_kv, d, ffn):
    """Shapes that are multiples of nothing: grouped heads, head sizes above and below a wave, odd widths."""
    w, m = variant(0, hidden=hidden, n_q=n_q, n_kv=n_kv, head_dim=d, ffn=ffn)
    run_case(w, m, [0, 37, 130, 16], block_bytes=64 << 10)


def test_fp32_three_layer_model_with_embedding_and_logits():
    w, m = variant(0, n_layers=3, vocab=777)
    lengths = [12, 100, 0, 77]
    case = DecodeCase(w, m, np.asarray(lengths, np.int32), full_model=True, block_bytes=64 << 10)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (4,))
    hid = case.run_gpu(token_ids=tok)
    ref_hid, ref_logits, ref_next = case.run_oracle(token_ids=tok)
    assert_close(hid, ref_hid, "hidden state", **F32_BAR)
    logits = case.logits_dev.cpu().numpy()
    assert_close(logits, ref_logits, "logits", **F32_BAR)
    case.check_cache(1e-4, 2e-5)
    nxt = case.next_dev.cpu().numpy()
    assert np.array_equal(nxt, np.argmax(logits, axis=-1))
    srt = np.sort(ref_logits, axis=-1)
    clear = (srt[:, -1] - srt[:, -2]) > 2e-4 * np.max(np.abs(ref_logits))
    assert np.array_equal(nxt[clear], ref_next[clear])


# ---- the other workloads at their real layer width (depth cut to what the oracle finishes in seconds) ----

def test_config2_width_two_layers_batch16_with_logits():
    """7B-class model, batch 16 at 1024 cached tokens, embedding + 2 of the 32 layers + output layer (V = 32000)."""
    w, m = variant(2, n_layers=2)
    lengths = wl.draw_lengths(w)
    assert len(lengths) == 16 and int(lengths[0]) == 1024
    case = DecodeCase(w, m, lengths, full_model=True)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (16,))
    hid = case.run_gpu(token_ids=tok)
    ref_hid, ref_logits, ref_next = case.run_oracle(token_ids=tok)
    assert_close(hid, ref_hid, "hidden state")
    logits = case.logits_dev.cpu().numpy()
    assert_close(logits, ref_logits, "logits")
    case.check_cache()
    nxt = case.next_dev.cpu().numpy()
    assert np.array_equal(nxt, np.argmax(logits, axis=-1))
    srt = np.sort(ref_logits, axis=-1)
    clear = (srt[:, -1] - srt[:, -2]) > 4e-2 * np.max(np.abs(ref_logits))
    assert np.array_equal(nxt[clear], ref_next[clear])


def test_config2_width_batch256():
    """The largest decode batch (one tile of 256 batch rows, no idle row) on one 7B-class layer."""
    w, m = variant(2, n_layers=1)
    run_case(w, m, [100 + (i * 37) % 400 for i in range(256)])


@pytest.mark.parametrize("n_q,n_kv,d,longest", [(4, 4, 64, 1500), (8, 2, 128, 1500), (7, 1, 128, 2700), (3, 3, 128, 1600)])
def test_uneven_lengths_with_a_list_of_chunks(n_q, n_kv, d, longest):
    """200 sequences, two of them long: the attention's grid follows the list of chunks that hold tokens (every kernel form, empty
    caches, whole and just begun chunks, two layers)."""
    lengths = np.asarray([(i * 7) % 45 for i in range(200)], np.int32)
    lengths[[3, 77, 199]] = longest, longest - 44, 255
    lengths[[10, 11, 12]] = 127, 128, 256
    w, m = variant(0, dtype="bf16", n_layers=2, hidden=256, n_q=n_q, n_kv=n_kv, head_dim=d, ffn=264)
    run_case(w, m, lengths)


@pytest.mark.parametrize("batch,vocab", [(34, 1003), (70, 1000), (130, 260), (200, 64), (256, 515)])
def test_output_layer_straight_from_the_tiles(batch, vocab):
    """Above 32 sequences, an output layer in one range of K: logits and argmax from the GEMM, every tile height, ragged last
    tiles and rows that are not 16-byte aligned.  Two equal rows of the output matrix give equal logits: the first maximum
    of every row is chosen."""
    def twins(case):
        wlm = case.extras_np["wlm"]
        wlm[vocab // 2 + 7:] = wlm[: vocab - vocab // 2 - 7]
    w, m = variant(0, dtype="bf16", n_layers=1, vocab=vocab)
    case = DecodeCase(w, m, np.asarray([3 + (i * 7) % 40 for i in range(batch)], np.int32), full_model=True, block_bytes=64 << 10, tweak=twins)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (batch,))
    case.run_gpu(token_ids=tok)
    _, ref_logits, _ = case.run_oracle(token_ids=tok)
    logits = case.logits_dev.cpu().numpy()
    assert_close(logits, ref_logits, "logits")
    assert (case.next_dev.cpu().numpy() == logits.argmax(1)).all()


def test_output_layer_straight_from_the_tiles_with_weights_read_once():
    """A step past the size of the caches and more weight tiles than compute units, at 40 and 200 sequences (the lowest and the
    tallest tile): the logits against the product of the same 16-bit operands in float64 -- fp32 sums of 1024 products, 1e-5 of
    the largest -- and the first maximum of every row."""
    w, m = variant(0, dtype="bf16", n_layers=1, hidden=1024, n_q=8, n_kv=8, head_dim=128, ffn=1024, vocab=131000)
    B, n_cu = 200, torch.cuda.get_device_properties(0).multi_processor_count
    assert -(-m.vocab // 256) > n_cu and 2 * (m.vocab * m.hidden + m.layer_params) > 256 << 20
    case = DecodeCase(w, m, np.asarray([3 + (i * 7) % 40 for i in range(B)], np.int32), full_model=True, block_bytes=256 << 10)
    tok = torch.from_numpy(wl.make_token_ids(dataclasses.replace(w, model=m), (B,)).astype(np.int32)).to(DEV)
    for batch in (40, 200):
        assert hb.dbg_decode_gemm_plan(batch, m.vocab, 1, m.hidden, n_cu, 192 << 20)["ksplit"] == 1
        case.slab.copy_(torch.from_numpy(case.img0.view(np.uint8)))
        y, nxt = torch.empty(batch, m.hidden, device=DEV), torch.empty(batch, dtype=torch.int32, device=DEV)
        logits = torch.full((batch, m.vocab), float("nan"), device=DEV)
        case.ctx.decode_step(batch=batch, kv_len=case.kv_len_dev, page_table=case.table_dev, max_pages=case.max_pages,
                             max_kv_len=int(case.kv_len.max()) + 1, token_ids=tok, logits=logits, next_token=nxt, x_out=y)
        torch.cuda.synchronize()
        case.ctx.check()
        x = y.double()
        rho = torch.rsqrt((x * x).mean(1, keepdim=True) + m.rms_eps)
        ref = rho * ((y * case.gf_dev).bfloat16().double() @ case.wlm_dev.double().t().contiguous())
        assert float((logits.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
        assert torch.equal(nxt.long(), torch.from_numpy(logits.cpu().numpy().argmax(1)).to(DEV))


@pytest.mark.parametrize("batch", [40, 100, 200])
def test_output_layer_in_ranges_of_k_with_unaligned_rows(batch):
    """The partial sums' own kernel, its stores element by element and the argmax in two passes: vocabulary 1003 in ranges of K."""
    w, m = variant(0, dtype="bf16", n_layers=1, hidden=1024, n_q=8, n_kv=8, head_dim=128, ffn=1024, vocab=1003)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    case = DecodeCase(w, m, np.asarray([3 + (i * 11) % 40 for i in range(batch)], np.int32), full_model=True, block_bytes=256 << 10)
    assert hb.dbg_decode_gemm_plan(batch, m.vocab, 1, m.hidden, n_cu, 192 << 20)["ksplit"] > 1
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (batch,))
    case.run_gpu(token_ids=tok)
    _, ref_logits, _ = case.run_oracle(token_ids=tok)
    logits = case.logits_dev.cpu().numpy()
    assert_close(logits, ref_logits, "logits")
    assert np.array_equal(case.next_dev.cpu().numpy(), np.argmax(logits, axis=-1))


@pytest.mark.parametrize("batch", [70, 150, 200])
def test_config4_width_batches_that_split_into_uneven_passes(batch):
    """Batches above 64 rows on the GQA layer: tiles of 128, 192 and 256 batch rows (70: 58 idle rows; 150: 42; 200: 56),
    every GEMM cut into ranges of K."""
    w, m = variant(4, n_layers=1)
    run_case(w, m, [60 + (i * 53) % 300 for i in range(batch)])


def test_config5_width_biases_at_batch_80():
    """The tiled path with q, k, v biases and groups of seven query heads per KV head (hidden 3584: 14 weight tiles of
    256 rows exactly; ffn 18944: 74)."""
    w, m = variant(5, n_layers=1)
    run_case(w, m, [40 + (i * 31) % 200 for i in range(80)])


def test_config3_width_layer_lognormal_lengths():
    """13B-class layer (hidden 5120, 40 heads, ffn 13824): 160 KiB pages do not divide the 2 MiB block (12 + slack),
    batch 32 with log-normal lengths capped at 4096."""
    w, m = variant(3, n_layers=1)
    lengths = wl.draw_lengths(w)
    case, stats = run_case(w, m, lengths)
    assert case.geom.pages_per_block == 12
    print("config 3 layer decode parity: max-abs ratio %.2e, rel-Fro %.2e, lengths %d..%d" % (stats + (lengths.min(), lengths.max())))


def test_config4_width_layer_gqa_long_context():
    """8B-class GQA layer (32 query / 8 KV heads, ffn 14336), batch 8, log-normal lengths capped at 8192."""
    w, m = variant(4, n_layers=1)
    lengths = wl.draw_lengths(w)
    case, stats = run_case(w, m, lengths)
    print("config 4 layer decode parity: max-abs ratio %.2e, rel-Fro %.2e, lengths %d..%d" % (stats + (lengths.min(), lengths.max())))


def test_config5_width_layer_biases_and_groups_of_seven():
    """Qwen2.5-7B-class layer (hidden 3584, 28 query / 4 KV heads, ffn 18944, RoPE base 1e6, biases on q, k, v), batch 8,
    log-normal lengths."""
    w, m = variant(5, n_layers=1)
    assert m.qkv_bias
    lengths = wl.draw_lengths(w)
    case, stats = run_case(w, m, lengths)
    assert "bq" in case.layers_np[0]
    print("config 5 layer decode parity: max-abs ratio %.2e, rel-Fro %.2e, lengths %d..%d" % (stats + (lengths.min(), lengths.max())))


def test_biases_small_shapes_bf16_and_fp32():
    """Biases with two layers, ragged lengths, both storage types (the fp32 path adds them in its rotary kernel)."""
    for dtype in ("bf16", "f32"):
        w, m = variant(0, dtype=dtype, n_layers=2, qkv_bias=True)
        run_case(w, m, [0, 5, 16, 31, 77])


@pytest.mark.parametrize("hidden,n_q,n_kv,d,ffn,lengths", [
    (256, 4, 4, 64, 688, [96]), (254, 6, 2, 64, 690, [0, 300]), (256, 2, 1, 96, 64, [255, 256, 257]),
    (510, 6, 3, 86, 130, [300, 0, 255, 77, 16, 511]), (130, 3, 1, 2, 34, [40, 1]), (64, 1, 1, 322, 48, [270, 3]),
    (130, 1, 1, 256, 33, [600, 1, 3, 17, 31]), (64, 2, 2, 320, 48, [5, 90, 16, 15, 2, 3, 7, 40, 520])])
def test_fp32_path_at_its_edges(hidden, n_q, n_kv, d, ffn, lengths):
    """The fp32 path over every number of batch rows a wave carries (1, 2, 4, 8, and a second tile of rows), contractions
    with and without 16-byte loads, head sizes of one to five lanes' elements, multiples of four and not, and blocks of 256 tokens; two layers, biases,
    embedding and logits."""
    w, m = variant(0, n_layers=2, hidden=hidden, n_q=n_q, n_kv=n_kv, head_dim=d, ffn=ffn, vocab=37, qkv_bias=True)
    lengths = np.asarray(lengths, np.int32)
    case = DecodeCase(w, m, lengths, full_model=True, block_bytes=64 << 10)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (len(lengths),))
    hid = case.run_gpu(token_ids=tok)
    ref_hid, ref_logits, _ = case.run_oracle(token_ids=tok)
    assert_close(hid, ref_hid, "hidden state", **F32_BAR)
    assert_close(case.logits_dev.cpu().numpy(), ref_logits, "logits", **F32_BAR)
    case.check_cache(1e-4, 2e-5)


def test_tiled_path_on_a_compute_unit_partition_and_in_a_replayed_graph():
    """The cut of the tiled GEMMs follows the compute units of the stream the step runs on (fewer ranges of K on a small
    partition): the result meets the oracle there too.  And the step is capturable: a replayed HIP graph gives the bits
    of the eager step on every replay, with eager work in between."""
    from paper_2511_11729_amd import colocate
    w, m = variant(0, dtype="bf16", n_layers=2, hidden=1024, n_q=8, n_kv=2, head_dim=128, ffn=2816, vocab=1000)
    lengths = np.asarray([5 + (i * 13) % 120 for i in range(100)], np.int32)
    case = DecodeCase(w, m, lengths, full_model=True, block_bytes=256 << 10)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (100,))
    ref_hid, ref_logits, _ = case.run_oracle(token_ids=tok)
    img0 = torch.from_numpy(case.img0.view(np.uint8))
    hid = case.run_gpu(token_ids=tok)
    assert_close(hid, ref_hid, "hidden state, whole chip")
    eager = (case.y_dev.clone(), case.logits_dev.clone(), case.slab.clone())
    cs = colocate.CuStreams()
    part = cs.low(2)                                   # 20 % of the compute units: other cuts
    case.slab.copy_(img0)
    torch.cuda.synchronize()
    hid_p = case.run_gpu(token_ids=tok, stream=part)
    assert_close(hid_p, ref_hid, "hidden state on 2/10 of the compute units")
    assert_close(case.logits_dev.cpu().numpy(), ref_logits, "logits on 2/10 of the compute units")
    case.check_cache()
    torch.cuda.synchronize()
    cs.close()
    # graph: captured on an ordinary stream, replayed three times with eager steps between the replays
    st = torch.cuda.Stream()
    tok_dev = torch.from_numpy(np.asarray(tok, np.int32)).to("cuda:0")
    y_g, logits_g, next_g = torch.empty_like(eager[0]), torch.empty_like(eager[1]), torch.empty_like(case.next_dev)

    def step():
        case.ctx.decode_step(batch=case.B, kv_len=case.kv_len_dev, page_table=case.table_dev, max_pages=case.max_pages,
                             max_kv_len=int(case.kv_len.max()) + 1, token_ids=tok_dev, logits=logits_g,
                             next_token=next_g, x_out=y_g, stream=st)

    case.slab.copy_(img0)
    torch.cuda.synchronize()
    step()
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        step()
    for rep in range(3):
        case.slab.copy_(img0)
        y_g.zero_()
        logits_g.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            g.replay()
        st.synchronize()
        assert torch.equal(y_g, eager[0]) and torch.equal(logits_g, eager[1]) and torch.equal(case.slab, eager[2])
        case.slab.copy_(img0)                          # the program's own eager work between replays
        torch.cuda.synchronize()
        case.run_gpu(token_ids=tok)
        assert torch.equal(case.y_dev, eager[0])
    case.ctx.check()
    del g


@pytest.mark.parametrize("batch", [4, 40])
def test_vocabulary_that_is_not_a_multiple_of_four(batch):
    """Rows of the logits that are not 16-byte aligned (vocabulary 1003) on both kernel families: the streaming output
    layer at batch 4, the tiled one at batch 40."""
    w, m = variant(0, dtype="bf16", n_layers=1, vocab=1003)
    lengths = np.asarray([3 + (i * 11) % 90 for i in range(batch)], np.int32)
    case = DecodeCase(w, m, lengths, full_model=True, block_bytes=64 << 10)
    tok = wl.make_token_ids(dataclasses.replace(w, model=m), (batch,))
    hid = case.run_gpu(token_ids=tok)
    ref_hid, ref_logits, _ = case.run_oracle(token_ids=tok)
    assert_close(hid, ref_hid, "hidden state")
    logits = case.logits_dev.cpu().numpy()
    assert_close(logits, ref_logits, "logits")
    assert np.array_equal(case.next_dev.cpu().numpy(), np.argmax(logits, axis=-1))


# (model, batch): weight tiles of 16 rows per matrix against 256 compute units choose how many tiles a wave takes
@pytest.mark.parametrize("idx,kw,batch", [
    (3, dict(ffn=13832), 9),                     # up to 16 rows: one tile per wave; 7 idle rows in the fragment
    (3, dict(ffn=13832), 17),                    # q,k,v 960 and gate/up 865 tiles (a ragged group of four): four; 320: two
    (5, dict(vocab=16 * 257 * 16 + 8), 12),      # an output layer of 4113 tiles above 8 rows: four, ragged
    (5, dict(vocab=1003), 32),                   # q,k,v 288, gate/up 1184 tiles: two; 224: one
])
def test_streaming_kernels_at_every_number_of_tiles_per_wave(idx, kw, batch):
    w, m = variant(idx, n_layers=1, **kw)
    lengths = np.asarray([(i * 23) % 70 for i in range(batch)], np.int32)
    full = "vocab" in kw
    case = DecodeCase(w, m, lengths, full_model=full)
    if full:
        tok = wl.make_token_ids(dataclasses.replace(w, model=m), (batch,))
        hid = case.run_gpu(token_ids=tok)
        ref_hid, ref_logits, _ = case.run_oracle(token_ids=tok)
        assert_close(case.logits_dev.cpu().numpy(), ref_logits, "logits")
    else:
        hid, ref_hid = case.run_gpu(), case.run_oracle()
    assert_close(hid, ref_hid, "hidden state")
    case.check_cache()


@pytest.mark.parametrize("batch", [2, 20, 40])
def test_an_infinite_value_element_stays_where_it_is(batch):
    """v is stored as it was computed, rotated with nothing: an infinite element (here through its bias) changes no other
    element of the appended vector, in particular not its rotation partner d/2 further."""
    w, m = variant(0, dtype="bf16", qkv_bias=True)
    lengths = np.asarray([3 + i % 20 for i in range(batch)], np.int32)
    images = []
    for value in (0.25, np.inf):
        def bias(case):
            case.layers_np[0]["bv"][5] = value
        case = DecodeCase(w, m, lengths, block_bytes=64 << 10, tweak=bias)
        case.run_gpu()
        images.append(case.slab_image())
    at = [case.geom.head_offset(int(case.table[b, n // 16]), 0, 1, 0, n % 16, m.head_dim * 2) // 2 + 5 for b, n in enumerate(lengths)]
    assert np.array_equal(np.flatnonzero(images[0] != images[1]), np.sort(at))
    assert np.all(images[1][at] == 0x7F80)                    # +infinity


@pytest.mark.parametrize("G", [4, 5, 8])
def test_a_key_with_an_infinite_element_takes_its_token_out(G):
    """A cached key element of -infinity against a query element that is positive in every head: the token's scores are
    -infinity, its probability is zero and the step is finite, on the vector and on the matrix units.  (The query element
    is the slowest rotation index under a large bias, so that no rotation changes its sign.)"""
    w, m = variant(0, dtype="bf16", hidden=G * 64, n_q=G, n_kv=1, head_dim=128, ffn=320, qkv_bias=True)

    def bias(case):
        case.layers_np[0]["bq"].reshape(G, 128)[:, 63] = 30.0
    case = DecodeCase(w, m, np.asarray([20, 150, 300], np.int32), block_bytes=64 << 10, tweak=bias)
    img = case.img0.copy()
    for b, n in enumerate(case.kv_len):                       # one token of each sequence, in its first, second or last chunk
        tok = (3, 140, 299)[b]
        img[case.geom.head_offset(int(case.table[b, tok // 16]), 0, 0, 0, tok % 16, 256) // 2 + 63] = 0xFF80
    case.img0 = img
    case.slab.copy_(torch.from_numpy(img.view(np.uint8)))
    y = case.run_gpu()
    assert_close(y, case.run_oracle(), "step with infinite keys")
