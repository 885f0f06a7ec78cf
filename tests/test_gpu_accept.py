"""GPU parity of psd_spec_accept against the CPU oracle, element by element on the same
seeded inputs.  Bar: accepted lengths and emitted tokens bit-exact given identical uniforms,
except at sequences where some tested position has |u - p/q| < 1e-5 (the oracle flags them;
they are counted and reported)."""
import numpy as np
import pytest
import torch

from oracle import accept as oacc
from paper_2510_26527_amd import runtime, synth
import paper_2510_26527_amd as psd

pytestmark = pytest.mark.gpu


def _to_f64(t):
    return t.detach().cpu().to(torch.float64).numpy()


def _compare(inp, temperature=1.0, n_p_rows=None):
    dev = torch.device("cuda")
    acc = runtime.Acceptor(dev)
    p, q, x, u = (inp[k].to(dev) for k in ("p", "q", "tokens", "uniforms"))
    n, tok, fl = acc(p, q, x, u, temperature)
    torch.cuda.synchronize()
    n, tok, fl = n.cpu().numpy().copy(), tok.cpu().numpy().copy(), fl.cpu().numpy().copy()
    T = float(np.float32(temperature))
    on, otok, ofl, rho = oacc.spec_accept(_to_f64(inp["p"]), _to_f64(inp["q"]), inp["tokens"].cpu().numpy(),
                                          _to_f64(inp["uniforms"]), T, return_rho=True)
    tie = (ofl & oacc.FLAG_NEAR_TIE) != 0
    len_mismatch = n != on
    assert not np.any(len_mismatch & ~tie), f"accept_len differs away from a near-tie: rows {np.nonzero(len_mismatch & ~tie)[0][:8]}"
    same = ~len_mismatch
    tok_mismatch = same & (tok != otok)
    assert not np.any(tok_mismatch), f"emitted token differs: rows {np.nonzero(tok_mismatch)[0][:8]}, gpu {tok[tok_mismatch][:8]} oracle {otok[tok_mismatch][:8]}"
    # the kernel's own near-tie flag covers every excused row
    assert np.all((fl[len_mismatch] & psd.PSD_FLAG_NEAR_TIE) != 0)
    # "the residual was empty, the draw used p" is reported for the same rows
    zr, ozr = (fl & psd.PSD_FLAG_ZERO_RESIDUAL) != 0, (ofl & oacc.FLAG_ZERO_RESIDUAL) != 0
    assert np.array_equal(zr[same], ozr[same]), f"zero-residual flag differs: rows {np.nonzero(same & (zr != ozr))[0][:8]}"
    assert np.all(n >= 0) and np.all(n <= inp["q"].shape[1])
    print(f"rows {len(n)}: near-tie rows {int(tie.sum())}, excused length flips {int(len_mismatch.sum())}, "
          f"mean accept_len {n.mean():.3f}")
    return n, tok, fl


@pytest.mark.parametrize("rows,gamma,V,dtype,bonus", [
    (5, 4, 1000, torch.bfloat16, True),        # one chunk, 16-byte aligned rows
    (3, 4, 1003, torch.bfloat16, True),        # V not a multiple of 8: scalar-load path
    (7, 3, 40000, torch.bfloat16, False),      # several chunks per row, ragged last chunk
    (4, 5, 20004, torch.float32, True),        # fp32 logits, several chunks
    (2, 1, 17, torch.float32, True),           # tiny vocabulary
    (1, 16, 8192, torch.float32, True),        # one sequence, long block
    (33, 2, 129, torch.float32, False),
])
def test_small_shapes(rows, gamma, V, dtype, bonus):
    inp = synth.make_accept_inputs(rows, gamma, V, seed=rows * 1000 + V, n_p_rows=gamma + (1 if bonus else 0), dtype=dtype)
    n, tok, _ = _compare(inp)
    if not bonus:
        assert np.all(tok[n == gamma] == -1)
    assert np.all(tok[n < gamma] >= 0)


@pytest.mark.parametrize("rows,gamma,V,dtype", [
    (1, 3, 512, torch.float32), (1, 3, 65536, torch.bfloat16), (1, 3, 65537, torch.float32), (60, 2, 4097, torch.float32),
    (130, 1, 4096, torch.bfloat16), (1, 2, 524289, torch.float32), (2, 5, 152065, torch.bfloat16)])
def test_draw_chunk_edges(rows, gamma, V, dtype):
    """The draw's division of the vocabulary: 512-entry chunks up to 128 of them, 4096-entry chunks at both sides of one,
    more than 128 chunks (larger ones), and more per-chunk statistics than eight lanes take in one round."""
    _compare(synth.make_accept_inputs(rows, gamma, V, seed=V + rows, n_p_rows=gamma + 1, dtype=dtype))


@pytest.mark.parametrize("rows,gamma,V,dtype", [
    (64, 1, 28672, torch.bfloat16), (64, 1, 28673, torch.float32), (40, 1, 65536, torch.float32), (40, 1, 65537, torch.bfloat16),
    (130, 1, 24584, torch.float32), (96, 1, 65544, torch.bfloat16), (96, 1, 57352, torch.bfloat16), (128, 1, 65536, torch.float32)])
def test_draw_quarters(rows, gamma, V, dtype):
    """The sums of a chunk's quarters kept one by one: whole chunks of 4096, a last chunk of one entry (three empty quarters), 64
    quarters and one chunk more (no quarters), chunks of 4096 with a short last one, of 8192 without quarters (65544: unaligned rows
    would need 68), of 8192 with a last one of 8 entries (57352) and whole ones (65536); draws that take each path at random."""
    _compare(synth.make_accept_inputs(rows, gamma, V, seed=V + rows, n_p_rows=gamma + 1, dtype=dtype))


@pytest.mark.parametrize("rows,gamma,V,dtype", [
    (8, 2, 16384, torch.float32), (8, 2, 16385, torch.bfloat16), (1, 3, 128256, torch.bfloat16), (2, 1, 262145, torch.float32),
    (128, 2, 8193, torch.float32), (103, 1, 10001, torch.float32), (96, 1, 40968, torch.bfloat16), (95, 1, 40968, torch.bfloat16), (96, 1, 40961, torch.float32)])
def test_draw_chunk_sizes(rows, gamma, V, dtype):
    """Both sides of each line of the division: 256 blocks of 512 entries, 512 blocks of 2048 (more than 128 of them a row,
    too), 96 sequences of more than 1024 chunks of 4096, aligned and not."""
    _compare(synth.make_accept_inputs(rows, gamma, V, seed=V + rows, n_p_rows=gamma + 1, dtype=dtype))



def test_workload2_full_size():
    """64 rows x gamma 8 x vocab 32000 bf16, the isolated acceptance workload, with and
    without the bonus row; mean accepted length lands near the 3.37 expected at alpha ~ 0.80."""
    for n_p in (8, 9):
        inp = synth.make_accept_inputs(64, 8, 32000, seed=2, n_p_rows=n_p, dtype=torch.bfloat16)
        n, tok, _ = _compare(inp)
        assert 2.3 < n.mean() < 4.5


def test_stress_shape_fp32_vocab_152064():
    inp = synth.make_accept_inputs(16, 16, 152064, seed=5, n_p_rows=17, dtype=torch.float32)
    _compare(inp)


def test_temperature():
    inp = synth.make_accept_inputs(16, 6, 5000, seed=9, n_p_rows=7, dtype=torch.float32)
    a = _compare(inp, temperature=0.7)
    b = _compare(inp, temperature=3.0)
    assert b[0].mean() >= a[0].mean()          # hotter -> flatter -> closer distributions


def test_degenerate_inputs():
    dev = torch.device("cuda")
    rows, gamma, V = 6, 4, 2048
    inp = synth.make_accept_inputs(rows, gamma, V, seed=4, n_p_rows=gamma + 1, dtype=torch.float32)
    # q == p: everything accepted, token is the bonus draw
    same = dict(inp); same["q"] = inp["p"][:, :gamma].clone()
    n, tok, fl = _compare(same)
    assert np.all(n == gamma) and np.all(tok >= 0)
    # draft token impossible under the target (-inf logit): rejected at position 0, even at u = 0
    hard = {k: v.clone() for k, v in inp.items()}
    hard["tokens"][:] = 3
    hard["p"][:, :, 3] = float("-inf")
    hard["uniforms"][:, 0] = 0.0
    n, tok, fl = _compare(hard)
    assert np.all(n == 0) and np.all(tok != 3)
    # gamma = 0 with one row: plain inverse-CDF sampling
    acc = runtime.Acceptor(dev)
    p = inp["p"][:, :1].contiguous().to(dev)
    u = inp["uniforms"][:, :1].contiguous().to(dev)
    n, tok, fl = acc(p, None, None, u, 1.0)
    torch.cuda.synchronize()
    ref = oacc.sample(_to_f64(inp["p"][:, 0]), _to_f64(inp["uniforms"][:, 0]))
    assert np.array_equal(tok.cpu().numpy(), ref) and np.all(n.cpu().numpy() == 0)


def _one_entry_apart(V, mass_log, direction, seed, rows=4):
    """q equals p except at one entry k per row whose probability under p is about exp(mass_log) and is doubled
    ("raised") or halved ("lowered") under q.  The draft token of position 0 is k when raised (ratio 1/2,
    rejected by u_0 = 0.75) and another token when lowered (ratio 1 - exp(mass_log)/2, rejected by the largest
    fp32 uniform below 1).  fp32 logits, gamma = 2, bonus row present."""
    rng = np.random.default_rng(seed)
    gamma = 2
    p = rng.normal(0.0, 2.0, (rows, gamma + 1, V)).astype(np.float32)
    q = p[:, :gamma].copy()
    k = rng.integers(0, V, rows)
    x = rng.integers(0, V, (rows, gamma)).astype(np.int32)
    u = rng.uniform(0.05, 0.95, (rows, gamma + 1)).astype(np.float32)
    for b in range(rows):
        lse = np.log(np.exp(p[b, 0].astype(np.float64)).sum())
        p[b, 0, k[b]] = np.float32(lse + mass_log)
        q[b, 0] = p[b, 0]
        q[b, 0, k[b]] = p[b, 0, k[b]] + np.float32(np.log(2.0) * (1 if direction == "raised" else -1))
        if direction == "raised":
            x[b, 0] = k[b]
            u[b, 0] = 0.75
        else:
            x[b, 0] = (k[b] + 1) % V
            u[b, 0] = np.nextafter(np.float32(1.0), np.float32(0.0))
    return {"p": torch.from_numpy(p), "q": torch.from_numpy(q), "tokens": torch.from_numpy(x),
            "uniforms": torch.from_numpy(u)}, k


def _draw_margin(inp, b):
    """Distance of u * (residual mass) from the nearest step of the residual's running sum at position 0 of row b,
    relative to the mass (numpy fp64; used only to keep the test's inputs away from a coin-flip draw)."""
    lp, lq = inp["p"][b, 0].double().numpy(), inp["q"][b, 0].double().numpy()
    pp = np.exp(lp - lp.max()); pp /= pp.sum()
    qq = np.exp(lq - lq.max()); qq /= qq.sum()
    r = np.maximum(pp - qq, 0.0)
    C = np.cumsum(r)
    t = float(inp["uniforms"][b, 2]) * r.sum()
    return np.abs(C - t).min() / r.sum(), r.sum()


@pytest.mark.parametrize("V", [3000, 40000])
def test_residual_support_q_equals_p_but_for_one_raised_entry(V):
    """Every other entry then has p_i - q_i = p_i (1 - Zp/Zq) > 0 by about 1e-9 p_i: a residual that exists only
    in fp64.  The emitted token and the zero-residual flag (not set: the residual is not empty) must be the
    oracle's."""
    inp, k = _one_entry_apart(V, np.log(1e-9), "raised", seed=V)
    # both sides compute these residual entries as differences of nearly equal numbers, good to ~1e-7 of their
    # size: keep each row's draw 100 times further than that from a step of the running sum
    rng = np.random.default_rng(V + 7)
    for b in range(inp["p"].shape[0]):
        for _ in range(200):
            margin, mass = _draw_margin(inp, b)
            assert 1e-10 < mass < 1e-8
            if margin >= 2e-5:
                break
            inp["uniforms"][b, 2] = float(rng.uniform(0.05, 0.95))
        assert margin >= 2e-5
    n, tok, fl = _compare(inp)
    assert np.all(n == 0) and np.all(tok != k)
    assert np.all((fl & psd.PSD_FLAG_ZERO_RESIDUAL) == 0)


@pytest.mark.parametrize("V", [3000, 40000])
def test_residual_support_q_equals_p_but_for_one_lowered_entry(V):
    """The residual is then the one lowered entry alone (every other p_i - q_i is negative by 5e-5 p_i); the
    rejection has to come from another token, whose ratio 1 - 5e-5 only the largest uniform below 1 rejects."""
    inp, k = _one_entry_apart(V, np.log(1e-4), "lowered", seed=V + 1)
    n, tok, fl = _compare(inp)
    assert np.all(n == 0) and np.array_equal(tok, k)
    assert np.all((fl & psd.PSD_FLAG_ZERO_RESIDUAL) == 0)


def test_strided_sequences_and_repeat_calls_are_deterministic():
    """p rows taken as a view of a larger logits buffer (a verify forward's output with extra
    leading rows): the sequence stride is larger than n_p_rows * V.  Two calls give identical
    results (no dependence on block scheduling)."""
    dev = torch.device("cuda")
    rows, gamma, V = 4, 5, 4096
    inp = synth.make_accept_inputs(rows, gamma, V, seed=12, n_p_rows=gamma + 1, dtype=torch.float32)
    big = torch.zeros((rows, gamma + 3, V), dtype=torch.float32, device=dev)
    big[:, 2:] = inp["p"].to(dev)
    acc = runtime.Acceptor(dev)
    q, x, u = inp["q"].to(dev), inp["tokens"].to(dev), inp["uniforms"].to(dev)
    outs = []
    for _ in range(3):
        n, tok, fl = acc(big[:, 2:], q, x, u, 1.0)
        torch.cuda.synchronize()
        outs.append((n.cpu().numpy().copy(), tok.cpu().numpy().copy()))
    on, otok, ofl = oacc.spec_accept(_to_f64(inp["p"]), _to_f64(inp["q"]), inp["tokens"].numpy(), _to_f64(inp["uniforms"]))
    ok = (ofl & 1) == 0
    assert np.array_equal(outs[0][0][ok], on[ok]) and np.array_equal(outs[0][1][ok], otok[ok])
    assert all(np.array_equal(outs[0][0], o[0]) and np.array_equal(outs[0][1], o[1]) for o in outs[1:])


# ---------------------------------------------------------------- greedy verification (temperature 0)
@pytest.mark.parametrize("rows,gamma,n_p,V,dtype", [
    (64, 8, 9, 32000, torch.bfloat16), (64, 8, 8, 32000, torch.bfloat16), (3, 5, 6, 1000, torch.float32),
    (16, 16, 17, 152064, torch.float32), (1, 10, 11, 128256, torch.float32), (7, 4, 5, 4099, torch.bfloat16),
    (5, 0, 1, 777, torch.float32), (2, 64, 65, 512, torch.bfloat16),
])
def test_greedy_matches_oracle_bit_exact(rows, gamma, n_p, V, dtype):
    """Greedy rule: drafts are the argmax of a noisy copy of p, so blocks end at every position.
    bf16 logits tie often (coarse values): the lowest-index rule is exercised on every row."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows * 1000 + gamma)
    p = torch.empty((rows, n_p, V), dtype=torch.float32, device="cuda").normal_(0, 2, generator=gen).to(dtype)
    noise = torch.empty((rows, gamma, V), dtype=torch.float32, device="cuda").normal_(0, 0.7, generator=gen)
    x = torch.argmax(p[:, :gamma].float() + noise, dim=-1).to(torch.int32)
    acc = runtime.Acceptor()
    n, tok, fl = acc(p, None, x, torch.empty((rows, gamma + 1), dtype=torch.float32, device="cuda"), 0.0)
    torch.cuda.synchronize()
    on, otok = oacc.greedy_accept(p.float().cpu().numpy(), x.cpu().numpy())
    assert np.array_equal(n.cpu().numpy(), on) and np.array_equal(tok.cpu().numpy(), otok)
    assert int(fl.abs().sum()) == 0
    if gamma >= 4 and rows >= 16:
        assert 0 < (on < gamma).mean() and on.max() > 0


def test_greedy_strided_rows_and_infinities():
    V, gamma = 1000, 3
    buf = torch.full((4, 6, V), float("-inf"), dtype=torch.float32, device="cuda")
    buf[:, :, 17] = 1.0
    buf[1, 2, 5] = 1.0                 # tie at position 2 of sequence 1: index 5 wins
    buf[2, 1, 900] = float("inf")
    p = buf[:, :4]                     # sequences 6*V apart, 4 rows used
    x = torch.tensor([[17, 17, 17], [17, 17, 17], [17, 17, 17], [17, 3, 17]], dtype=torch.int32, device="cuda")
    acc = runtime.Acceptor()
    n, tok, _ = acc(p, None, x, torch.empty((4, gamma + 1), device="cuda"), 0.0)
    torch.cuda.synchronize()
    on, otok = oacc.greedy_accept(p.cpu().numpy(), x.cpu().numpy())
    assert n.cpu().tolist() == on.tolist() == [3, 2, 1, 1]
    assert tok.cpu().tolist() == otok.tolist() == [17, 5, 900, 17]


def test_edge_sizes():
    """One-entry vocabulary (every ratio is 1, every draw is token 0), the longest block the boundary accepts
    (gamma = 64), and rows = 0 (a no-op that launches nothing)."""
    dev = torch.device("cuda")
    acc = runtime.Acceptor(dev)
    one = {"p": torch.randn(3, 3, 1), "q": torch.randn(3, 2, 1), "tokens": torch.zeros((3, 2), dtype=torch.int32),
           "uniforms": synth.make_uniforms((3, 3), 1)}
    n, tok, _ = _compare(one)
    assert np.all(n == 2) and np.all(tok == 0)
    inp = synth.make_accept_inputs(3, 64, 300, seed=64, n_p_rows=65, dtype=torch.float32, noise_std=0.1)
    n, tok, _ = _compare(inp)
    assert n.max() > 8
    empty = torch.empty((0, 3, 16), dtype=torch.float32, device=dev)
    ws = torch.empty(256, dtype=torch.uint8, device=dev)
    psd.psd_spec_accept(empty, empty[:, :2], torch.empty((0, 2), dtype=torch.int32, device=dev), 2,
                        torch.empty((0, 3), dtype=torch.float32, device=dev), 1.0,
                        torch.empty(0, dtype=torch.int32, device=dev), torch.empty(0, dtype=torch.int32, device=dev),
                        0, 3, 16, psd.PSD_F32, 48, 32, None, ws)
    torch.cuda.synchronize()
