"""GPU: projections over more than 64 rows, which run the LDS-tiled GEMM or, where few
workgroups and a short K leave that behind, the streaming layouts in 64-row blocks; at the
edges of tiles and K slices, against the oracle: prompts one row past a tile count, models
whose row tiles do not fill a workgroup, an FFN width that leaves half a 64-column chunk
(int8, Q4_0), every tile shape of the tiled kernel."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_logits_close, build_pair, dev_i32, gpu_logits, gpu_step

pytestmark = pytest.mark.gpu


def _bound(ref):
    """K and V are rounded to fp16 once per layer (2^-11 of a value); a value that passed two
    layers carries at most four such roundings of the largest value beside it."""
    return 4 * 2.0 ** -11 * np.abs(ref[np.isfinite(ref)]).max()

# 688 = 21.5 x 32 columns of the down projection; 43 row tiles of gate/up pairs
RAGGED = synth.SMALL_BF16
# grouped-query heads and biases; 1504 = 47 x 32 columns (an odd count of 32-column steps)
GQA = dataclasses.replace(synth.SMALL_MQA, d_ff=1504)


@pytest.mark.parametrize("dtype", ["bf16", "w8", "q4"])
@pytest.mark.parametrize("shape,n", [(RAGGED, 65), (RAGGED, 257), (GQA, 129), (GQA, 300)],
                         ids=["ragged65", "ragged257", "gqa129", "gqa300"])
def test_prompt_rows_and_next_step(dtype, shape, n):
    """The prompt's K/V in every layer and the next step's logits."""
    import torch
    import paper_2606_13740_amd as dl

    model, om, _ = build_pair(shape, dtype, max_window=64, max_pos=n + 64)
    kv = dl.KVCache(model, n + 64)
    prompt = synth.prompt_ids(shape, n)
    dl.dllm_prefill(model.handle, kv.handle, dev_i32(prompt), n)
    torch.cuda.synchronize()
    okv = oracle.OracleKV(shape, n + 64)
    oracle.prefill(om, okv, prompt)
    K, Vt = (t.cpu().numpy().astype(np.float64) for t in kv.views())
    for l in range(shape.n_layers):
        rk, rv = okv.K[l, :n].transpose(1, 0, 2), okv.V[l, :n].transpose(1, 0, 2)
        assert np.abs(K[l][:, :n] - rk).max() <= _bound(rk)
        assert np.abs(Vt[l][:, :, :n].transpose(0, 2, 1) - rv).max() <= _bound(rv)
    tok, mask = synth.window(shape, 32, range(8, 32))
    got, _, _ = gpu_logits(model, kv, tok, mask)
    ref = oracle.denoise_step(om, okv, tok, mask)
    assert_logits_close(got, ref.logits, _bound(ref.logits))
    kv.close()
    model.close()


@pytest.mark.parametrize("dtype", ["bf16", "w8", "q4"])
@pytest.mark.parametrize("W", [65, 96, 131, 256])
def test_wide_window(dtype, W):
    """Windows past 64 rows after a prompt (every row sees every key; per-row limits and explicit
    positions past 64 rows are in test_gpu_merged)."""
    import paper_2606_13740_amd as dl

    shape = RAGGED
    model, om, _ = build_pair(shape, dtype, max_window=256, max_pos=512)
    kv = dl.KVCache(model, 40 + W)
    prompt = synth.prompt_ids(shape, 40)
    dl.dllm_prefill(model.handle, kv.handle, dev_i32(prompt), 40)
    okv = oracle.OracleKV(shape, 40 + W)
    oracle.prefill(om, okv, prompt)
    tok, mask = synth.window(shape, W, range(W // 3, W))
    got, _, _ = gpu_logits(model, kv, tok, mask)
    ref = oracle.denoise_step(om, okv, tok, mask)
    assert_logits_close(got, ref.logits, _bound(ref.logits))
    kv.close()
    model.close()


def test_long_prompt_attention_head_64():
    """32 heads of 64: a prompt long enough for two query tiles per wave whose last row group is
    half empty (its second layer's K/V depend on them), then steps whose key splits are long
    enough for three staging buffers, or (9 rows) two to a CU."""
    import paper_2606_13740_amd as dl

    shape = synth.Shape(n_layers=2, d_model=2048, n_heads=32, head_dim=64, d_ff=256, vocab=500, mask_id=499)
    n = 2850
    model, om, _ = build_pair(shape, "bf16", max_window=64, max_pos=n + 64)
    kv = dl.KVCache(model, n + 64)
    prompt = synth.prompt_ids(shape, n)
    dl.dllm_prefill(model.handle, kv.handle, dev_i32(prompt), n)
    okv = oracle.OracleKV(shape, n + 64)
    oracle.prefill(om, okv, prompt)
    for W in (9, 17, 33, 64):
        tok, mask = synth.window(shape, W, range(4, W))
        got, _, _ = gpu_logits(model, kv, tok, mask)
        ref = oracle.denoise_step(om, okv, tok, mask)
        assert_logits_close(got, ref.logits, _bound(ref.logits))
    kv.close()
    model.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("head_dim,n_kv,n", [(64, 0, 2048 + 1), (64, 0, 2304 - 63), (128, 4, 2048 + 1)])
def test_two_tile_prompt_rows(head_dim, n_kv, n):
    """Two layers, so that the second layer's K/V depend on the two-tile attention of every row."""
    import torch
    import paper_2606_13740_amd as dl

    shape = synth.Shape(n_layers=2, d_model=32 * head_dim, n_heads=32, head_dim=head_dim, d_ff=256, vocab=500,
                        mask_id=499, n_kv_heads=n_kv)
    model, om, _ = build_pair(shape, "bf16", max_window=64, max_pos=n)
    kv = dl.KVCache(model, n)
    prompt = synth.prompt_ids(shape, n)
    dl.dllm_prefill(model.handle, kv.handle, dev_i32(prompt), n)
    torch.cuda.synchronize()
    okv = oracle.OracleKV(shape, n)
    oracle.prefill(om, okv, prompt)
    K, Vt = (t.cpu().numpy().astype(np.float64) for t in kv.views())
    rk, rv = okv.K[1, :n].transpose(1, 0, 2), okv.V[1, :n].transpose(1, 0, 2)
    assert np.abs(K[1][:, :n] - rk).max() <= _bound(rk)
    assert np.abs(Vt[1][:, :, :n].transpose(0, 2, 1) - rv).max() <= _bound(rv)
    kv.close()
    model.close()


def _second_layer_kv(shape, dtype, n):
    """(K, V) of layer 1 after an n-row prompt, on the GPU and from the oracle."""
    import torch
    import paper_2606_13740_amd as dl

    model, om, _ = build_pair(shape, dtype, max_window=64, max_pos=n)
    kv = dl.KVCache(model, n)
    prompt = synth.prompt_ids(shape, n)
    dl.dllm_prefill(model.handle, kv.handle, dev_i32(prompt), n)
    torch.cuda.synchronize()
    okv = oracle.OracleKV(shape, n)
    oracle.prefill(om, okv, prompt)
    K, Vt = (t.cpu().numpy().astype(np.float64) for t in kv.views())
    kv.close()
    model.close()
    return ((K[1][:, :n], okv.K[1, :n].transpose(1, 0, 2)),
            (Vt[1][:, :, :n].transpose(0, 2, 1), okv.V[1, :n].transpose(1, 0, 2)))


@pytest.mark.parametrize("dtype", ["bf16", "w8", "q4"])
@pytest.mark.parametrize("d_ff,n", [(4000, 257), (4000, 401), (8016, 257), (12048, 257), (4000, 769), (16016, 257)],
                         ids=["6x8", "8x8", "12x8", "12x16", "16x8", "16x16"])
def test_tile_shapes(dtype, d_ff, n):
    """Gate/up in each tile shape, the last workgroup of rows and of tokens not full, and (int8 and
    Q4_0 at d_ff 16016, bf16 always) down in eight K slices of 500 or more columns."""
    shape = synth.Shape(n_layers=2, d_model=256, n_heads=2, head_dim=128, d_ff=d_ff, vocab=500, mask_id=499)
    print(f"case: tile shapes, {dtype}, d_ff {d_ff}, {n} rows", flush=True)
    for got, ref in _second_layer_kv(shape, dtype, n):
        assert np.abs(got - ref).max() <= _bound(ref)


@pytest.mark.parametrize("dtype", ["bf16", "w8", "q4"])
@pytest.mark.parametrize("n", [128, 256, 300])
def test_qkv_on_both_sides_of_the_layout_rule(dtype, n):
    """160 row tiles of QKV (heads of 64, grouped): one round of streaming workgroups up to 256
    rows, the tiled kernel in K slices after, and O and down of 80 tiles on either."""
    shape = synth.Shape(n_layers=2, d_model=1280, n_heads=20, head_dim=64, d_ff=1504, vocab=500, mask_id=499,
                        n_kv_heads=10, qkv_bias=True)
    print(f"case: layout rule, {dtype}, {n} rows", flush=True)
    for got, ref in _second_layer_kv(shape, dtype, n):
        assert np.abs(got - ref).max() <= _bound(ref)


@pytest.mark.parametrize("dtype", ["bf16", "w8", "q4"])
def test_results_do_not_depend_on_earlier_calls(dtype):
    """A 100-row prompt and a 96-row window on a new model, and again after a 600-row prompt has
    grown its workspace: the same bits in the cache, the ids and the confidences."""
    import torch
    import paper_2606_13740_amd as dl

    shape = RAGGED
    model, _, _ = build_pair(shape, dtype, max_window=96, max_pos=640, oracle_too=False)
    tok, mask = synth.window(shape, 96, range(30, 96))

    def once():
        kv = dl.KVCache(model, 196)
        dl.dllm_prefill(model.handle, kv.handle, dev_i32(synth.prompt_ids(shape, 100)), 100)
        ids, conf = gpu_step(model, kv, tok, mask)
        out = kv.buf.cpu().numpy(), ids, conf
        kv.close()
        return out

    before = once()
    kv = dl.KVCache(model, 600)
    dl.dllm_prefill(model.handle, kv.handle, dev_i32(synth.prompt_ids(shape, 600)), 600)
    torch.cuda.synchronize()
    kv.close()
    for a, b in zip(before, once()):
        np.testing.assert_array_equal(a, b)
    model.close()
