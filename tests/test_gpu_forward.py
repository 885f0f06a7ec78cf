"""GPU parity of psd_model_forward / psd_kv_truncate against the CPU oracle on the same
seeded weights, KV contents and tokens.  Bars: fp32 models max-abs logit error <= 1e-4;
bf16 models, per logits row, max|gpu - oracle| / max|oracle| <= 2e-2."""
import os
import time

import numpy as np
import pytest
import torch

from oracle import forward as ofwd
from paper_2510_26527_amd import runtime, synth
import paper_2510_26527_amd as psd

pytestmark = pytest.mark.gpu

F32_ABS_TOL = 1e-4
BF16_REL_TOL = 2e-2


def _progress(msg):
    """Long tests append to a progress file so that a quiet run is not mistaken for a hang."""
    os.makedirs("gpurun_out", exist_ok=True)
    with open("gpurun_out/test_progress.log", "a") as f:
        f.write(f"{time.strftime('%H:%M:%S')} {msg}\n")
    print(msg, flush=True)


def check_logits(gpu, ref, dtype, what=""):
    gpu = gpu.detach().cpu().double().numpy().reshape(-1, ref.shape[-1])
    ref = ref.reshape(-1, ref.shape[-1])
    assert np.all(np.isfinite(gpu)), f"{what}: non-finite logits"
    err = np.abs(gpu - ref).max(axis=1)
    if dtype == torch.float32:
        assert err.max() <= F32_ABS_TOL, f"{what}: max abs err {err.max():.3e}"
        return err.max()
    rel = err / np.abs(ref).max(axis=1)
    assert rel.max() <= BF16_REL_TOL, f"{what}: max rel err {rel.max():.3e}"
    return rel.max()


class Pair:
    """The same model, cache contents and lengths on both sides."""

    def __init__(self, shape, dtype, batch, max_len, seed=0, ctx=None, lens=None, std=0.02, oracle_kv_dtype=np.float64,
                 oracle_rows=None, pack=False, share=None, w4=False):
        self.shape, self.dtype, self.batch = shape, dtype, batch
        self.w = synth.make_weights(shape, seed, dtype, std=std, share=share)
        if w4:
            # 4-bit projections: the GPU gets codes + scales + zero points, the oracle the dequantised matrices
            from oracle import quant as oquant
            codes, quant = synth.quantize_w4(self.w)
            self.model = runtime.Model(shape, codes, quant=quant)
            self.w = {k: (torch.from_numpy(oquant.dequantize(codes[k].numpy(), quant[k][0].float().numpy(),
                                                               quant[k][1].numpy())) if k in quant else v)
                      for k, v in self.w.items()}
            pack = True
        else:
            self.model = runtime.Model(shape, self.w)
        if pack:
            self.model.pack()
        self.kv = runtime.KVCache(self.model, batch, max_len, fill_garbage=True)
        self.cfg = ofwd.ModelConfig(**shape.asdict())
        self.rows = list(range(batch)) if oracle_rows is None else oracle_rows   # sequences the oracle follows
        self.okv = ofwd.KVCache(self.cfg, len(self.rows), max_len, oracle_kv_dtype)
        if ctx:
            lens = [ctx] * batch if lens is None else lens
            ks, vs = synth.make_kv_fill(shape, batch, ctx, seed + 1, dtype)
            self.kv.load(ks, vs, lens)
            for l in range(shape.n_layers):
                self.okv.k[l][:, :, :ctx] = ofwd.widen(ks[l][self.rows])
                self.okv.v[l][:, :, :ctx] = ofwd.widen(vs[l][self.rows])
            self.okv.lens = np.array([lens[b] for b in self.rows], np.int64)

    def step(self, tokens, n_logit_rows=None, what=""):
        tokens = np.asarray(tokens, np.int32)
        t = torch.from_numpy(tokens).cuda()
        out = runtime.forward(self.model, self.kv, t, n_logit_rows)
        torch.cuda.synchronize()
        ref = ofwd.forward(self.cfg, self.w, tokens[self.rows], self.okv)
        if n_logit_rows == 0:
            return None
        if n_logit_rows is not None:
            ref = ref[:, -n_logit_rows:]
        return check_logits(out[self.rows], ref, self.dtype, what)

    def close(self):
        self.kv.close()
        self.model.close()


@pytest.mark.parametrize("shape", [synth.TINY_TARGET, synth.TINY_INTERMEDIATE, synth.TINY_DRAFT],
                         ids=["target", "intermediate", "draft"])
def test_fp32_tiny_models(shape):
    """Workload 1's three models: 31-token prefill, then verify-shaped steps of 9, 5, 1 and 2 rows."""
    p = Pair(shape, torch.float32, 1, 128, seed=11)
    toks = synth.make_tokens(shape.vocab, (1, 48), 3)
    p.step(toks[:, :31], 0)
    e = [p.step(toks[:, 31:40], what="9 rows"), p.step(toks[:, 40:45], what="5 rows"),
         p.step(toks[:, 45:46], what="1 row"), p.step(toks[:, 46:48], what="2 rows")]
    print("max abs logit error", max(e))
    p.close()


def test_fp32_batch_with_ragged_lengths_and_truncate():
    shape = synth.TINY_INTERMEDIATE
    p = Pair(shape, torch.float32, 3, 64, seed=5, ctx=20, lens=[20, 7, 13], std=0.05)
    toks = synth.make_tokens(shape.vocab, (3, 14), 8)
    p.step(toks[:, :6], what="6 rows")
    # roll back to base + keep + 1 per sequence on the device, mirror it in the oracle
    base = torch.tensor([20, 7, 13], dtype=torch.int32, device="cuda")
    keep = torch.tensor([5, 0, 2], dtype=torch.int32, device="cuda")
    psd.psd_kv_truncate(p.kv.handle, base, keep, 1, 26)
    p.okv.truncate([26, 8, 16])
    torch.cuda.synchronize()
    assert p.kv.lens.cpu().tolist() == [26, 8, 16] and psd.psd_kv_len_upper_bound(p.kv.handle) == 26
    p.step(toks[:, 6:14], what="after truncate")
    # truncation never lengthens
    psd.psd_kv_truncate_to(p.kv.handle, 1000)
    torch.cuda.synchronize()
    assert p.kv.lens.cpu().tolist() == [34, 16, 24]
    psd.psd_kv_truncate_to(p.kv.handle, 10)
    torch.cuda.synchronize()
    assert p.kv.lens.cpu().tolist() == [10, 10, 10] and psd.psd_kv_len_upper_bound(p.kv.handle) == 10
    p.close()


def step_launches(p, *args, **kwargs):
    """One checked step, and how often each kind of kernel was launched: which path a call took."""
    psd.psd_profile_enable(1000)
    p.step(*args, **kwargs)
    counts = {kind: n for kind, (_, n) in psd.psd_profile_collect().items()}
    psd.psd_profile_enable(0)
    return counts


SMALL_GQA = synth.Shape(2, 256, 4, 2, 64, 512, 1024, 1.0e4)           # d_head 64, group 2
SMALL_MHA = synth.Shape(2, 256, 2, 2, 128, 384, 1000, 1.0e4)          # d_head 128, ragged vocab tiles
SMALL_G7 = synth.Shape(1, 896, 7, 1, 128, 1152, 2048, 1.0e6)          # Qwen2-like group of 7


@pytest.mark.parametrize("d_model,batch,n_new,rows", [(128, 1, 1, 1), (128, 1, 8, 8), (128, 2, 5, 3), (384, 1, 16, 16), (128, 2, 20, 1), (4224, 1, 2, 2)])
def test_head_in_whole_tiles(d_model, batch, n_new, rows):
    """A head of up to 16 rows whose whole tiles fill the chip writes the logits and moves the lengths itself: folded and not, a
    subset of the rows, from a pass of more than 16 rows (no row scale), a ragged last tile, more than 256 sums of squares a row
    (d_model 4224)."""
    shape = synth.Shape(1, d_model, d_model // 64, d_model // 64, 64, 128, 29505, 1.0e4)
    p = Pair(shape, torch.bfloat16, batch, 64, seed=n_new, ctx=9, std=0.05, pack=True)
    ran = step_launches(p, synth.make_tokens(shape.vocab, (batch, n_new), d_model), n_logit_rows=rows, what="the last rows' logits")
    assert ran["gemm_reduce"] == 0 and ran["lens"] == 0
    assert p.kv.lens.cpu().tolist() == [9 + n_new] * batch
    p.close()


@pytest.mark.parametrize("batch,n_new,rows,vocab", [(2, 20, 4, 200), (3, 9, 3, 29505), (1, 300, 16, 200)])
def test_head_over_few_rows_of_a_long_pass(batch, n_new, rows, vocab):
    """The up to 16 rows with logits of a longer pass reach the packed head in operand order, one sequence's behind the other's: up
    to 8 rows (folded) and more, from the norm of up to 256 rows and above."""
    shape = synth.Shape(1, 128, 2, 2, 64, 128, vocab, 1.0e4)
    p = Pair(shape, torch.bfloat16, batch, 320, seed=n_new, ctx=9, std=0.05, pack=True)
    p.step(synth.make_tokens(shape.vocab, (batch, n_new), rows), n_logit_rows=rows, what="the last rows' logits")
    assert p.kv.lens.cpu().tolist() == [9 + n_new] * batch
    p.close()


@pytest.mark.parametrize("d_head", [64, 128])
def test_staged_attention_in_operand_order(d_head):
    """Packed pass of 16 rows whose LDS-staged attention has more than 64 query rows per KV head and one split of the cache, so that it
    writes the operand order itself."""
    shape = synth.Shape(1, 8 * d_head, 8, 1, d_head, 256, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 64, seed=d_head, ctx=20, std=0.05, pack=True)
    p.step(synth.make_tokens(shape.vocab, (1, 16), 3), what="16 rows x 8 heads")
    p.close()


@pytest.mark.parametrize("n_new", [17, 33, 64, 65, 97, 128])
@pytest.mark.parametrize("d_model,d_ffn,vocab", [(128, 11008, 28001), (128, 14336, 40960), (384, 18944, 512), (1024, 512, 41600)])
def test_rows_kernel(d_model, d_ffn, vocab, n_new):
    """17 to 128 rows on packed weights, every number of 16-row tiles (2, 3, 4, 6, 8) at one of its edges: gate | up with its SwiGLU in
    whole tiles of 6 strips, the last one half there (11008), of 8 (14336) and of 10 (18944; 65 rows and more: LDS-tiled); up to 64
    rows heads in whole tiles of 8 strips with a ragged last one (28001), of 10 (40960) and in shared tiles (41600 at K = 1024); one K
    step and three, so that a block is through before its ring of four steps turns."""
    shape = synth.Shape(1, d_model, d_model // 64, d_model // 64, 64, d_ffn, vocab, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 192, seed=n_new, ctx=20, std=0.05, pack=True)
    ran = step_launches(p, synth.make_tokens(shape.vocab, (1, n_new), d_ffn), what="all rows' logits")
    most = {11008: 96, 14336: 128, 18944: 64, 512: 0}[d_ffn]              # rows up to which gate | up is in whole tiles
    assert ran["swiglu"] == (0 if n_new <= most else 1)
    if n_new <= 64 and vocab > 512:
        assert ran["gemm_reduce"] == (1 if vocab == 41600 else 0)
    p.close()


@pytest.mark.parametrize("d_model,d_ffn,vocab,n_new", [
    (1024, 11008, 28001, 17), (1024, 11008, 28001, 65), (1024, 11008, 28001, 96), (1024, 14336, 32000, 65), (1024, 14336, 32000, 128),
    (1024, 18944, 40960, 33), (1024, 18944, 40960, 64), (128, 28672, 512, 45), (1024, 28672, 128256, 17), (1024, 28672, 128256, 64)])
def test_rows_kernel_walks_its_ring(d_model, d_ffn, vocab, n_new):
    """Eight K steps and more: a block's ring of four steps turns, for 6, 8 and 10 strips, gate | up and head, and 2 to 8 row tiles; and
    blocks of several whole tiles, the next one requested while this one is multiplied: two of gate | up (28672, of one K step and of
    eight), four of a head (128256)."""
    shape = synth.Shape(1, d_model, d_model // 64, d_model // 64, 64, d_ffn, vocab, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 192, seed=n_new, ctx=20, std=0.02, pack=True)
    ran = step_launches(p, synth.make_tokens(shape.vocab, (1, n_new), d_ffn), what="all rows' logits")
    assert ran["swiglu"] == 0 and (vocab == 512 or ran["gemm_reduce"] == 0)
    p.close()


def test_rows_kernel_shares_tiles_of_three_segments():
    """Q, K and V of 33 tiles each, shared by all blocks: a block goes on from one segment to the next in the middle of its range."""
    shape = synth.Shape(1, 4224, 66, 66, 64, 128, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 128, seed=4, ctx=20, std=0.02, pack=True)
    p.step(synth.make_tokens(shape.vocab, (1, 50), 6), what="50 rows")
    p.close()


@pytest.mark.parametrize("hq,hk,batch,n_new,ctx", [(1, 1, 1, 130, 0), (3, 1, 2, 70, 9), (8, 2, 1, 200, 33), (7, 1, 2, 75, 0), (5, 1, 1, 129, 100), (2, 2, 2, 700, 0),
                                                    (32, 32, 1, 258, 0), (64, 16, 1, 140, 372), (32, 32, 8, 130, 670)])
def test_attention_of_a_prompt(hq, hk, batch, n_new, ctx):
    """Blocks of 128 query rows that walk the keys their rows see, longest first: one and several query heads per KV head, fewer blocks
    than heads in the group (70 rows), blocks that reach into the next head's rows, heads of several blocks with some left over, ragged
    lengths; enough rows (8 192 with the heads) over up to 512 keys for one split; and so many heads on so many keys (256 on 800) that each
    head's blocks stay side by side."""
    shape = synth.Shape(1, 128, hq, hk, 128, 128, 200, 1.0e4)
    lens = [ctx - 8 * b for b in range(batch)] if ctx else None
    p = Pair(shape, torch.bfloat16, batch, (ctx + n_new + 63) // 64 * 64, seed=n_new, ctx=ctx, lens=lens, std=0.05,
             oracle_rows=[0, batch - 1] if batch > 2 else None)
    p.step(synth.make_tokens(shape.vocab, (batch, n_new), hq), what="all rows' logits")
    p.close()


@pytest.mark.parametrize("heads,vocab,n_new,rows", [(2, 48900, 300, 300), (32, 512, 1500, 1), (32, 512, 2200, 1)])
def test_tiles_of_two_widths(heads, vocab, n_new, rows):
    """A projection of which a first launch does whole rounds of wide tiles and a second the other columns in narrower ones: a head
    with a ragged last tile; Q, K and V with the line inside V (1500 rows) and inside K, all of V behind it (2200).  Scores have a spread of std^2 d_model; a score at four times that, with
    its factors in bf16, moves its probability by 4 std^2 d_model 2^-9: 0.6 % at 0.02, 4 % at 0.05, past the tolerance."""
    shape = synth.Shape(1, 2048, heads, heads, 128, 128, vocab, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 2304, seed=n_new, ctx=0, std=0.02)
    ran = step_launches(p, synth.make_tokens(shape.vocab, (1, n_new), heads), n_logit_rows=rows, what="the logits")
    assert ran["gemm_tiled"] == (6 if rows > 1 else 5)          # four projections, the long pass' head, and one launch more
    p.close()


@pytest.mark.parametrize("n_new", [1, 8, 9, 16])
@pytest.mark.parametrize("d_model,d_ffn", [(128, 128), (384, 1408), (256, 5760), (256, 4224)])
def test_operand_order_activations(d_model, d_ffn, n_new):
    """Activations between the packed projections of up to 16 rows, folded (8 rows) and not (9), 1 and 16 rows: K of fewer 32-k
    quarters than the column kernel has wavefronts (128, 256), of a few each (384, 1408), and of one round of its loads, folded
    (11: 5760) or not (8: 4224), and a little more."""
    shape = synth.Shape(1, d_model, d_model // 64, d_model // 64, 64, d_ffn, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 128, seed=n_new, ctx=40, std=0.05, pack=True)
    toks = synth.make_tokens(shape.vocab, (1, n_new + 3), d_ffn)
    p.step(toks[:, :n_new], what="all rows' logits")
    p.step(toks[:, n_new:], n_logit_rows=1, what="the last row's")
    p.close()


@pytest.mark.parametrize("n_new", [1, 8, 9, 16, 17])
@pytest.mark.parametrize("d_model,hq,hk,d_ffn", [
    (128, 2, 2, 128), (384, 2, 1, 4224), (128, 44, 22, 11008), (256, 64, 32, 14464), (128, 80, 40, 18944), (640, 64, 64, 24448), (128, 2, 2, 28544)])
def test_projections_in_bands(d_model, hq, hk, d_ffn, n_new):
    """QKV and gate|up by bands: gate bands of 1 to 7 strips, whole and with a last one of fewer; QKV in bands of 3 (the last one not full),
    4, 5 and 6 strips, or, narrow, on shared tiles; one, two, three and five K steps for two groups of wavefronts; folded (8 rows) and not.
    17 rows: the rows kernel on the same packed copies of gate|up (of QKV in these few steps of K the tiled kernel; the next test has more)."""
    shape = synth.Shape(1, d_model, hq, hk, 128, d_ffn, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 64, seed=n_new, ctx=9, std=0.02, pack=True)
    ran = step_launches(p, synth.make_tokens(shape.vocab, (1, n_new), d_ffn), what="all rows' logits")
    if n_new <= 16:
        assert ran["swiglu"] == 0 and ran["gemm_skinny"] == 3
    p.close()


@pytest.mark.parametrize("n_new", [16, 17, 45, 64])
@pytest.mark.parametrize("d_model,hq,hk", [(4096, 32, 32), (3840, 44, 22), (2944, 58, 29), (2176, 78, 39), (1792, 64, 64), (512, 60, 60)])
def test_rows_kernel_reads_bands(d_model, hq, hk, n_new):
    """QKV in bands of 3, 3, 4, 5 and 6 strips, read by the rows kernel in tiles of eight strips that blocks share: tiles that begin in the middle of a
    band, bands (of 3 and 5) that hold the end of Q and the beginning of K, a last one that is not full; and bands of 6 in whole tiles of 6.
    16 rows: the band kernel itself."""
    shape = synth.Shape(1, d_model, hq, hk, 128, 128, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 128, seed=n_new, ctx=20, std=0.02, pack=True)
    ran = step_launches(p, synth.make_tokens(shape.vocab, (1, n_new), hq), n_logit_rows=3, what="three rows' logits")
    assert n_new > 16 or ran["gemm_skinny"] == 3
    p.close()


@pytest.mark.parametrize("n_new", [1, 8, 9, 16])
@pytest.mark.parametrize("d_model,d_ffn", [(4224, 128), (4224, 1152), (128, 16384)])
def test_down_projection_by_units(d_model, d_ffn, n_new):
    """The down projection of wide models, and of a d_ffn seven times as long, on the unit kernel: every tile by one block (66 tiles of
    one K step), shared unevenly (66 of 9 steps by 256 blocks), and by 128 blocks each (2 of 128); folded (8 rows) and not.  The
    second step finds the arrival counters as the first left them.  A score at four times its spread std^2 d_model, with its factors in
    bf16, moves its probability by 4 std^2 d_model 2^-9: 1.3 % at 0.02 and 4224, 8 % at 0.05, past the tolerance."""
    shape = synth.Shape(2, d_model, 2, 2, 64, d_ffn, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 128, seed=n_new, ctx=40, std=0.02, pack=True)
    toks = synth.make_tokens(shape.vocab, (1, 2 * n_new), d_ffn)
    p.step(toks[:, :n_new], what="all rows' logits")
    p.step(toks[:, n_new:], n_logit_rows=1, what="the last row's")
    p.close()


@pytest.mark.parametrize("shape,n_new,ctx", [
    (SMALL_GQA, 1, 300), (SMALL_GQA, 5, 200), (SMALL_GQA, 8, 300), (SMALL_GQA, 9, 1000), (SMALL_GQA, 17, 129), (SMALL_GQA, 40, 64),
    (SMALL_MHA, 8, 1024), (SMALL_MHA, 11, 77), (SMALL_MHA, 70, 200), (SMALL_MHA, 130, 0), (SMALL_MHA, 200, 30),
    (SMALL_GQA, 170, 0),
    (SMALL_G7, 16, 520), (SMALL_G7, 17, 4096), (SMALL_G7, 3, 5),
])
@pytest.mark.parametrize("pack", [False, True], ids=["rowmajor", "packed"])
def test_bf16_small_models(shape, n_new, ctx, pack):
    """Both weight layouts of the M <= 16 path (row-major split-K kernel, packed stream-K kernels).
    Covers the skinny GEMM at 1-3 row tiles, the tiled GEMM (70, 130 rows: 128-row blocks; 170, 200 rows: 256-row
    blocks with two sets of LDS tiles), ragged N and M,
    attention on both sides of the switch between its two kernels (10 and 11 query rows per KV head), with 1, 2 and 4
    query tiles, several query chunks (7 x 17 rows), split counts from 1 to 17 and a prefill with an empty cache.  std 0.05 keeps the signal above bf16 noise."""
    max_len = (ctx + n_new + 70 + 63) // 64 * 64
    p = Pair(shape, torch.bfloat16, 1, max_len, seed=n_new, ctx=ctx or None, std=0.05, pack=pack)
    toks = synth.make_tokens(shape.vocab, (1, n_new + 6), n_new + ctx)
    e1 = p.step(toks[:, :n_new], what="first step")
    e2 = p.step(toks[:, n_new:], n_logit_rows=4, what="second step, last 4 rows")
    print("rel err", e1, e2)
    p.close()


@pytest.mark.parametrize("rows", [17, 64, 65, 128, 129, 256, 257, 301])
@pytest.mark.parametrize("w4", [False, True], ids=["bf16", "w4"])
def test_tiled_projections_at_tile_edges(rows, w4):
    """Row counts around the tile heights (64, 128, 256), output widths that no tile divides (384 + 2 x 128 columns of
    QKV, 777 of the head), K of 3 and 128 K tiles (shared unevenly by the blocks), and from 129 rows on a gate|up
    projection wide enough (2 x 16384) to apply SwiGLU itself.  Bar: the repository's 2e-2 for bf16 models."""
    shape = synth.Shape(1, 384, 3, 1, 128, 8192 if rows > 256 or rows < 129 else 16384, 777, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 320, seed=70 + rows, std=0.05, w4=w4)
    p.step(synth.make_tokens(shape.vocab, (1, rows), rows), what=f"{rows} rows")
    p.close()


@pytest.mark.parametrize("rows,d,ffn,vocab", [(65, 256, 640, 500), (128, 384, 1024, 777), (127, 2560, 2560, 900),
                                               (40, 128, 256, 65537), (64, 256, 256, 65600), (100, 256, 384, 65700),
                                               (20, 512, 512, 65700), (64, 512, 512, 65700)])
def test_tiled_projections_of_small_products_and_wide_heads(rows, d, ffn, vocab):
    """65 to 128 rows on 64-row tiles (few K tiles) next to products on 128-row tiles (2560 x 7680: 2560 of them), and heads
    of 512 column tiles and more, given out whole, the last one a part, or (20 rows of d_model 512) shared."""
    shape = synth.Shape(1, d, d // 64, d // 64, 64, ffn, vocab, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 192, seed=rows, std=0.05)
    p.step(synth.make_tokens(vocab, (1, rows), rows), what=f"{rows} rows")
    p.close()


@pytest.mark.parametrize("d_head,batch,rows", [(128, 2, 15), (64, 3, 16), (128, 3, 17), (64, 2, 33), (128, 1, 65)])
def test_rotation_and_append_at_tile_edges(d_head, batch, rows):
    """Steps of more than 10 query rows per KV head, which the rotation kernel prepares: row counts around its 16-row
    value tiles, several sequences at ragged positions, 3 + 1 query and key heads (a part of one block's), split counts
    that are no multiple of the four in flight; a second step reads what the first appended."""
    shape = synth.Shape(1, 384, 384 // d_head, 1, d_head, 640, 500, 1.0e4)
    lens = [130 - 9 * b for b in range(batch)]
    p = Pair(shape, torch.bfloat16, batch, 320, seed=rows, ctx=130, lens=lens, std=0.05)
    toks = synth.make_tokens(shape.vocab, (batch, rows + 12), rows)
    p.step(toks[:, :rows], what="first step")
    p.step(toks[:, rows:], what="second step")
    p.close()


@pytest.mark.parametrize("d_head,batch,ctx,rows", [(128, 40, 300, 3), (64, 40, 300, 10), (128, 24, 700, 1), (64, 130, 70, 2)])
def test_attention_of_many_sequences(d_head, batch, ctx, rows):
    """More 256-key splits than CUs: the build of the direct attention kernel that runs two blocks per CU on 32-key
    tiles, with ragged lengths (from one key on), several splits and, at 130 x 4 heads, a single one."""
    shape = synth.Shape(1, 256, 4, 4, d_head, 256, 600, 1.0e4)
    lens = [1 + (ctx - 1) * ((7 * b) % batch) // batch for b in range(batch - 1)] + [ctx]
    p = Pair(shape, torch.bfloat16, batch, (ctx + 2 * rows + 63) // 64 * 64, seed=batch, ctx=ctx, lens=lens, std=0.05)
    toks = synth.make_tokens(shape.vocab, (batch, 2 * rows), 5)
    p.step(toks[:, :rows], what="first step")
    p.step(toks[:, rows:], what="second step")
    p.close()


@pytest.mark.parametrize("d_head,batch,ctx,rows", [(64, 50, 700, 2), (128, 64, 330, 3), (128, 40, 100, 3), (64, 43, 129, 1)])
def test_attention_of_one_split_per_head(d_head, batch, ctx, rows):
    """Two blocks per CU and one split of the cache, the step's own rows riding on it: 172 to 256 heads at any length, 160
    heads with at most 128 keys (129 keys and 172 heads: one; the second step is past 128 keys)."""
    shape = synth.Shape(1, 256, 4, 4, d_head, 256, 600, 1.0e4)
    lens = [1 + (ctx - 1) * ((7 * b) % batch) // batch for b in range(batch - 1)] + [ctx]
    p = Pair(shape, torch.bfloat16, batch, (ctx + 2 * rows + 63) // 64 * 64, seed=batch, ctx=ctx, lens=lens, std=0.05)
    toks = synth.make_tokens(shape.vocab, (batch, 2 * rows), 5)
    p.step(toks[:, :rows], what="first step")
    p.step(toks[:, rows:], what="second step")
    p.close()


def test_workspace_covers_every_cache_length():
    """16 sequences x 4 KV heads: a 900-key step takes more, shorter key splits than one at the end of its 1408-key cache;
    the workspace that the cache's size asks for has to serve it."""
    shape = synth.Shape(1, 256, 4, 4, 64, 256, 600, 1.0e4)
    p = Pair(shape, torch.bfloat16, 16, 1408, seed=3, ctx=896, std=0.05)
    need = psd.psd_model_workspace_bytes(p.model.handle, 16, 3, 1408)
    assert need > 0
    p.step(synth.make_tokens(shape.vocab, (16, 3), 5), what="896 keys")
    p.close()


def test_bf16_batch_ragged_lengths_truncate():
    shape = SMALL_GQA
    p = Pair(shape, torch.bfloat16, 4, 640, seed=21, ctx=512, lens=[512, 100, 333, 1], std=0.05, pack=True)
    toks = synth.make_tokens(shape.vocab, (4, 33), 2)
    p.step(toks[:, :16], what="16 rows x 4 sequences")
    base = torch.tensor([512, 100, 333, 1], dtype=torch.int32, device="cuda")
    keep = torch.tensor([16, 0, 7, 3], dtype=torch.int32, device="cuda")
    psd.psd_kv_truncate(p.kv.handle, base, keep, 0)          # bound argument left out: the host bound stays
    assert psd.psd_kv_len_upper_bound(p.kv.handle) == 528
    p.okv.truncate([528, 100, 340, 4])
    p.step(toks[:, 16:33], what="17 rows after truncate")
    torch.cuda.synchronize()
    assert p.kv.lens.cpu().tolist() == [545, 117, 357, 21]
    p.close()


def test_batched_verify_loop_with_per_sequence_rollback_only():
    """Fourteen consecutive verify steps of 16 sequences near the end of their caches: forward over gamma + 1
    rows, acceptance against a synthetic drafter, then psd_kv_truncate alone (no psd_kv_truncate_to), the way a
    decoding loop runs: it reads the accepted lengths back to steer itself and hands the largest resulting length
    to the rollback.  Every step's logits and every acceptance are compared with the oracle.  A host bound that
    only ever grew by gamma + 1 per step would pass the cache size after eleven steps and refuse the rest."""
    from oracle import accept as oacc
    shape, B, gamma, max_len, steps = SMALL_GQA, 16, 7, 384, 14
    rng = np.random.default_rng(3)
    lens0 = [int(v) for v in rng.integers(260, 300, B)]
    p = Pair(shape, torch.bfloat16, B, max_len, seed=31, ctx=300, lens=lens0, std=0.05, pack=True)
    acc = runtime.Acceptor("cuda")
    lens = np.array(lens0)
    assert psd.psd_kv_len_upper_bound(p.kv.handle) == lens.max()
    assert lens.max() + steps * (gamma + 1) > max_len
    total_kept = 0
    for it in range(steps):
        toks = synth.make_tokens(shape.vocab, (B, gamma + 1), 100 + it)
        t = torch.from_numpy(toks).cuda()
        base = torch.from_numpy(lens.astype(np.int32)).cuda()
        logits = runtime.forward(p.model, p.kv, t)
        ref = ofwd.forward(p.cfg, p.w, toks, p.okv)
        check_logits(logits, ref, torch.bfloat16, f"step {it}")
        q, _ = synth.make_draft_from_target(logits[:, :gamma], 1.0, 200 + it)
        x = t[:, 1:].contiguous()                       # the rows after x* verify the tokens fed after it
        u = synth.make_uniforms((B, gamma + 1), 300 + it, "cuda")
        n, tok, fl = acc(logits, q, x, u, 1.0)
        keep = n.cpu().numpy().astype(np.int64)         # the loop's one read-back per step
        lens = lens + 1 + keep
        psd.psd_kv_truncate(p.kv.handle, base, n, 1, int(lens.max()))
        torch.cuda.synchronize()
        on, otok, ofl = oacc.spec_accept(logits.cpu().double().numpy(), q.cpu().double().numpy(), x.cpu().numpy(),
                                         u.cpu().double().numpy())
        ok = (ofl & oacc.FLAG_NEAR_TIE) == 0
        assert np.array_equal(keep[ok], on[ok]) and np.array_equal(tok.cpu().numpy()[ok], otok[ok])
        total_kept += int(keep.sum())
        p.okv.truncate([int(v) for v in lens])
        assert p.kv.lens.cpu().tolist() == [int(v) for v in lens]
        assert psd.psd_kv_len_upper_bound(p.kv.handle) == lens.max()
    assert 0 < total_kept < steps * B * gamma
    p.close()


def test_outputs_and_scratch_stay_inside_their_buffers():
    """Canaries around everything the calls write: logits, the forward workspace (sized by the library's own
    answer), the acceptance outputs and workspace.  A kernel that writes one element past its buffer flips one."""
    dev = torch.device("cuda")
    guard, mark = 1024, -12345.0
    for shape, n_new, ctx, pack in ((SMALL_GQA, 8, 300, True), (SMALL_MHA, 11, 77, False), (SMALL_G7, 17, 520, True),
                                    (SMALL_MHA, 70, 200, False)):
        w = synth.make_weights(shape, 9, torch.bfloat16, std=0.05)
        model = runtime.Model(shape, w)
        if pack:
            model.pack()
        max_len = (ctx + n_new + 63) // 64 * 64
        kv = runtime.KVCache(model, 1, max_len)
        ks, vs = synth.make_kv_fill(shape, 1, ctx, 10, torch.bfloat16)
        kv.load(ks, vs, ctx)
        need = psd.psd_model_workspace_bytes(model.handle, 1, n_new, max_len)
        ws_all = torch.full((need // 4 + 2 * guard,), mark, dtype=torch.float32, device=dev)
        ws = ws_all[guard:guard + need // 4].view(torch.uint8)
        assert ws.data_ptr() % 256 == 0
        lg_all = torch.full((n_new * shape.vocab + 2 * guard,), mark, dtype=torch.float32, device=dev)
        logits = lg_all[guard:guard + n_new * shape.vocab].view(1, n_new, shape.vocab)
        toks = torch.from_numpy(synth.make_tokens(shape.vocab, (1, n_new), 5)).to(dev)
        psd.psd_model_forward(model.handle, toks, n_new, kv.handle, logits, n_new, ws)
        torch.cuda.synchronize()
        for name, t, n in (("workspace", ws_all, need // 4), ("logits", lg_all, n_new * shape.vocab)):
            assert bool((t[:guard] == mark).all()) and bool((t[guard + n:] == mark).all()), f"{name} guard touched ({shape}, {n_new})"
        assert bool(torch.isfinite(logits).all())
        # acceptance on these logits
        gamma = min(n_new - 1, 16)
        q, x = synth.make_draft_from_target(logits[:, :gamma], 0.5, 3)
        u = synth.make_uniforms((1, gamma + 1), 4, dev)
        a_need = psd.psd_spec_accept_workspace_bytes(1, gamma, gamma + 1, shape.vocab)
        aw_all = torch.full((a_need // 4 + 2 * guard,), mark, dtype=torch.float32, device=dev)
        aw = aw_all[guard:guard + a_need // 4].view(torch.uint8)
        out_all = torch.full((3 + 2 * 64,), -777, dtype=torch.int32, device=dev)
        out = out_all[64:67]
        psd.psd_spec_accept(logits, q, x, gamma, u, 1.0, out[0:1], out[1:2], 1, gamma + 1, shape.vocab, psd.PSD_F32,
                            n_new * shape.vocab, gamma * shape.vocab, out[2:3], aw)
        torch.cuda.synchronize()
        assert bool((aw_all[:guard] == mark).all()) and bool((aw_all[guard + a_need // 4:] == mark).all())
        assert bool((out_all[:64] == -777).all()) and bool((out_all[67:] == -777).all())
        assert 0 <= int(out[0]) <= gamma
        kv.close()
        model.close()


def test_forward_is_deterministic():
    shape = SMALL_MHA
    w = synth.make_weights(shape, 3, torch.bfloat16, std=0.05)
    model = runtime.Model(shape, w).pack()
    toks = torch.from_numpy(synth.make_tokens(shape.vocab, (2, 9), 1)).cuda()
    outs = []
    for _ in range(3):
        kv = runtime.KVCache(model, 2, 1088)
        ks, vs = synth.make_kv_fill(shape, 2, 1024, 7, torch.bfloat16)
        kv.load(ks, vs, 1024)
        outs.append(runtime.forward(model, kv, toks).clone())
        kv.close()
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    model.close()


def test_capacity_error_is_raised_on_the_host():
    shape = synth.TINY_DRAFT
    p = Pair(shape, torch.float32, 1, 64, seed=1)
    toks = synth.make_tokens(shape.vocab, (1, 70), 1)
    p.step(toks[:, :60], 0)
    with pytest.raises(psd.PsdError) as e:
        runtime.forward(p.model, p.kv, torch.from_numpy(toks[:, 60:70]).cuda())
    assert e.value.status == psd.PSD_ERR_CAPACITY
    p.close()


def test_workload3_llama2_7b_full_size():
    """Workload 3 at full size: LLaMA2-7B shape, bf16, 8 new tokens on a 1024-token N(0,1) cache.
    Then the 9-row variant after a rollback to 1024 + 3 accepted."""
    shape = synth.LLAMA2_7B
    _progress("w3: generating 7B weights")
    p = Pair(shape, torch.bfloat16, 1, 1088, seed=3, ctx=1024, oracle_kv_dtype=np.float32, pack=True)
    toks = synth.make_tokens(shape.vocab, (1, 17), 33)
    _progress("w3: forward 8 rows, both sides")
    e1 = p.step(toks[:, :8], what="8 rows")
    psd.psd_kv_truncate_to(p.kv.handle, 1027)
    p.okv.truncate(1027)
    _progress(f"w3: rel err {e1:.3e}; forward 9 rows after rollback")
    e2 = p.step(toks[:, 8:17], what="9 rows")
    _progress(f"w3: rel err {e2:.3e}")
    p.close()


def test_workload5_qwen2_7b_full_size_sampled_sequences():
    """Workload 5 at full size on the GPU (16 sequences, 16 new rows, 4096-token caches); the
    oracle follows sequences 0 and 11 only (its attention and GEMM rows are independent per
    sequence), which bounds its time."""
    shape = synth.QWEN2_7B
    _progress("w5: generating Qwen2-7B-shaped weights and 16 x 4096 caches")
    p = Pair(shape, torch.bfloat16, 16, 4160, seed=5, ctx=4096, oracle_kv_dtype=np.float32, oracle_rows=[0, 11])
    toks = synth.make_tokens(shape.vocab, (16, 16), 55)
    _progress("w5: forward 16 x 16 rows")
    e = p.step(toks, n_logit_rows=16, what="16x16 rows")
    _progress(f"w5: rel err {e:.3e}")
    p.close()


def test_workload4_chain_models_full_size():
    """Workload 4's three models at full size, each at the row count its verify step has in the
    chain (gamma_intermediate + 1 = 11 rows for the LLaMA3-8B-shaped target: 44 query rows per KV
    head; gamma_draft + 1 = 7 rows for the intermediate with d_head 64; 1 and 2 rows for the
    one-layer draft that shares the target's embedding and lm_head), against 300-token caches."""
    _progress("w4: generating LLaMA3-8B-shaped target")
    tgt = Pair(synth.LLAMA3_8B, torch.bfloat16, 1, 384, seed=41, ctx=300, oracle_kv_dtype=np.float32, pack=True)
    toks = synth.make_tokens(synth.LLAMA3_8B.vocab, (1, 14), 44)
    _progress("w4: target forward 11 rows, both sides")
    e = tgt.step(toks[:, :11], what="target 11 rows")
    _progress(f"w4: target rel err {e:.3e}")
    share = {"embed": tgt.w["embed"], "lm_head": tgt.w["lm_head"]}
    drf = Pair(synth.CHAIN_DRAFT, torch.bfloat16, 1, 384, seed=43, ctx=300, oracle_kv_dtype=np.float32, pack=True,
               share=share)
    assert drf.model.weights["lm_head"].data_ptr() != 0
    e1 = drf.step(toks[:, :1], what="draft 1 row")
    e2 = drf.step(toks[:, 1:3], what="draft 2 rows")
    _progress(f"w4: draft rel err {e1:.3e} {e2:.3e}")
    drf.close()
    tgt.close()
    del drf, tgt, share
    mid = Pair(synth.CHAIN_INTERMEDIATE, torch.bfloat16, 1, 384, seed=42, ctx=300, oracle_kv_dtype=np.float32,
               pack=True)
    e = mid.step(toks[:, :7], what="intermediate 7 rows")
    _progress(f"w4: intermediate rel err {e:.3e}")
    mid.close()


@pytest.mark.parametrize("shape,steps,ctx", [
    (SMALL_GQA, (1, 8, 16, 3), 300), (SMALL_MHA, (9, 16), 77), (SMALL_G7, (5, 11), 520), (SMALL_GQA, (16, 16, 16), 0),
])
def test_w4_small_models(shape, steps, ctx):
    """4-bit weight-only quantised projections (the format of the paper's intermediate model): steps of 1 to 16
    rows, with and without cached context, against the oracle run on the dequantised weights."""
    max_len = (ctx + sum(steps) + 17 + 63) // 64 * 64
    p = Pair(shape, torch.bfloat16, 1, max_len, seed=ctx + 1, ctx=ctx or None, std=0.05, w4=True)
    toks = synth.make_tokens(shape.vocab, (1, sum(steps)), ctx + 2)
    at, errs = 0, []
    for n in steps:
        errs.append(p.step(toks[:, at:at + n], what=f"{n} rows"))
        at += n
    print("w4 rel err", errs)
    p.close()


@pytest.mark.parametrize("n_new", [1, 9, 16])
@pytest.mark.parametrize("d_model,d_ffn", [(128, 128), (640, 2176), (256, 14336), (4224, 384), (128, 16384)])
def test_w4_projections_with_one_owner_per_output(d_model, d_ffn, n_new):
    """4-bit O and down by strips: one K step for sixteen wavefronts (128), 5 and 17, and 112 (7 each, a burst of four and one of three);
    down, and for a wide model O too, by units (4224; 16384 against 128); gate|up by tiles of 64 columns over K of one quad that is
    not full, of one and a quarter, and of more."""
    shape = synth.Shape(2, d_model, 2, 1, 64, d_ffn, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 64, seed=n_new, ctx=20, std=0.02, w4=True)
    toks = synth.make_tokens(shape.vocab, (1, n_new + 2), d_ffn)
    ran = step_launches(p, toks[:, :n_new], what="all rows' logits")
    assert ran["swiglu"] == 0
    p.step(toks[:, n_new:], n_logit_rows=1, what="the last row's")
    p.close()


@pytest.mark.parametrize("n_new", [1, 16])
@pytest.mark.parametrize("d_ffn", [128, 1152])
def test_w4_gate_up_in_ranges(d_ffn, n_new):
    """4-bit gate|up of a wide model whose tiles leave most CUs idle (2 and 18 of them, K of ten quads): equal ranges of K in partial slots, the
    row scale and SwiGLU where they are added."""
    shape = synth.Shape(2, 5120, 2, 1, 64, d_ffn, 200, 1.0e4)
    p = Pair(shape, torch.bfloat16, 1, 64, seed=n_new, ctx=20, std=0.02, w4=True)
    ran = step_launches(p, synth.make_tokens(shape.vocab, (1, n_new), d_ffn), what="all rows' logits")
    assert ran["swiglu"] == 2
    p.close()


def test_w4_more_than_16_rows():
    """More than 16 rows in one call run on the tiled kernel with the 4-bit weights dequantised on their way into
    LDS: a long step of one sequence (a prompt), logits for the trailing rows only or for all of them, then steps of
    several ragged sequences at 18 and 160 rows (both block heights of the tiled kernel), and back to a short step."""
    shape = SMALL_GQA
    p = Pair(shape, torch.bfloat16, 1, 256, seed=77, ctx=40, std=0.05, w4=True)
    toks = synth.make_tokens(shape.vocab, (1, 86), 5)
    e1 = p.step(toks[:, :37], what="37 rows, all logits")
    e2 = p.step(toks[:, 37:70], n_logit_rows=21, what="33 rows, last 21 logits")
    e3 = p.step(toks[:, 70:86], what="16 rows after the long steps")
    print("w4 long steps rel err", e1, e2, e3)
    assert int(p.kv.lens[0]) == 126 and psd.psd_kv_len_upper_bound(p.kv.handle) == 126
    p.close()
    p2 = Pair(shape, torch.bfloat16, 2, 128, seed=78, ctx=10, lens=[10, 3], std=0.05, w4=True)
    assert psd.psd_model_workspace_bytes(p2.model.handle, 2, 9, 128) > 0
    toks = synth.make_tokens(shape.vocab, (2, 12), 6)
    e4 = p2.step(toks[:, :9], what="2 sequences x 9 rows")
    e5 = p2.step(toks[:, 9:12], what="2 sequences x 3 rows after it")
    p2.close()
    p3 = Pair(SMALL_G7, torch.bfloat16, 8, 128, seed=79, ctx=50, lens=[50, 1, 33, 17, 40, 8, 25, 49], std=0.05, w4=True)
    toks = synth.make_tokens(SMALL_G7.vocab, (8, 20), 7)
    e6 = p3.step(toks, n_logit_rows=2, what="8 sequences x 20 rows, last 2 logits rows")
    print("w4 batched long steps rel err", e4, e5, e6)
    p3.close()


def test_w4_batch_of_sequences():
    p = Pair(SMALL_GQA, torch.bfloat16, 4, 448, seed=8, ctx=384, lens=[384, 10, 200, 77], std=0.05, w4=True)
    toks = synth.make_tokens(SMALL_GQA.vocab, (4, 8), 5)
    p.step(toks[:, :4], what="4 sequences x 4 rows")
    p.step(toks[:, 4:8], n_logit_rows=2, what="4 x 4 rows, last 2 logits rows")
    p.close()


def test_w4_llama3_8b_full_size():
    """The paper's intermediate at full size: a 4-bit, group-128 copy of the LLaMA3-8B-shaped target, 11 rows
    (gamma_intermediate + 1) on a 300-token cache and then 20 rows in one step, against the oracle on the dequantised
    weights."""
    _progress("w4: generating and quantising LLaMA3-8B-shaped weights")
    p = Pair(synth.LLAMA3_8B, torch.bfloat16, 1, 384, seed=41, ctx=300, oracle_kv_dtype=np.float32, w4=True)
    toks = synth.make_tokens(synth.LLAMA3_8B.vocab, (1, 31), 44)
    _progress("w4: forward 11 rows, both sides")
    e = p.step(toks[:, :11], what="w4 target 11 rows")
    _progress(f"w4: rel err {e:.3e}")
    # 20 more rows in one step: the projections dequantise the caller's codes on their way into the tiled kernel
    _progress("w4: forward 20 rows, both sides")
    e = p.step(toks[:, 11:], n_logit_rows=4, what="w4 target 20 rows, last 4 logits rows")
    _progress(f"w4: rel err at 20 rows {e:.3e}")
    p.close()
