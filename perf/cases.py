"""The work whose time this repository is measured by: batched Transformer execution through the model entry points
(Model.encode, Model.decode_step, Model.seq_release), from the smallest model at four short prompts to full-width
layers of the three large shapes.

A case names a model shape of `workload` (or a generic shape with 64-wide heads), how many of its layers run, a batch
with the distribution of its input lengths, and what one pass does:

  phase "job"     encode the batch, run `steps` decode iterations, release it.  The prompt-heavy cases take one iteration,
                  which reads the keys and values that the encode call left behind
  phase "decode"  one decode iteration of a live batch.  The batch grows by a position per pass, as it does in service;
                  when a sequence reaches the end of its reservation the batch is replaced by the prompts again

The tokens fed to decode iterations are given (drawn from the seed), not the ones just generated, so that two
implementations whose logits differ in the last bit go on with the same inputs.  Outputs are the logits of every call
(hidden states for a model without an embedding, the encoder output too for an encoder-decoder model).  The greedy tokens
are asked for, as a serving loop does, but not returned: they are the argmax of the returned rows, and near ties go
either way.
"""
import numpy as np
import torch

import paper_2404_07947_amd as exe
import workload as wl

DEV = "cuda:0"


def _head64_shape(dtype):
    """A generic decoder-only model with 64-wide heads: 16 heads, hidden 1024, feed-forward 4096."""
    return wl.tiny_shape().replace(name="head64", n_layers=6, d_model=1024, n_heads=16, d_ff=4096, vocab=32000, max_pos=2048,
                                   dtype=dtype)


def _shape(case):
    L = case["layers"]
    f32 = case["dtype"] == "f32"
    dt = wl.DTYPE_F32 if f32 else wl.DTYPE_BF16
    if case["model"] == "tiny":
        return wl.tiny_shape().replace(n_layers=L, max_pos=1024, dtype=dt)
    if case["model"] == "small_t5":
        return wl.small_t5_shape(dt).replace(n_layers=L, n_dec_layers=L)
    if case["model"] == "head64":
        return _head64_shape(dt).replace(n_layers=L)
    if case["model"] == "opt13b":
        return wl.opt13b_shape(L)
    if case["model"] == "t5_11b":
        return wl.t5_11b_shape(case["enc_layers"], L)
    return wl.gpt3_175b_share_shape(L)


def _case(model, dtype, layers, phase, batch, mean, std, lo, hi, steps=0, block=0, enc_layers=0):
    return {"model": model, "dtype": dtype, "layers": layers, "enc_layers": enc_layers, "phase": phase, "batch": batch,
            "mean": mean, "std": std, "lo": lo, "hi": hi, "steps": steps, "block": block}


def listed():
    named = {
        # The smallest job: four prompts of 8 to 32 tokens in float, then 16 decode iterations; a pass is 17 calls, each
        # a few microseconds of arithmetic, so launches and host work count.
        "tiny_job": _case("tiny", "f32", 2, "job", 4, 20, 7, 8, 32, steps=16),
        # A small encoder-decoder model in float: ragged inputs, self- and cross-attention with relative-position bias.
        "t5_small_job": _case("small_t5", "f32", 2, "job", 12, 96, 48, 8, 200, steps=20),
        # Long prompts through the float path: the precision a user checks a model in before serving it in bf16.
        "tiny_encode_f32": _case("tiny", "f32", 2, "job", 32, 384, 128, 64, 1000, steps=1),
        # Head size 64 in bf16 (half of the supported head sizes): a batch of prompts, and a job most of which is decoding, on a
        # paged pool.
        "head64_encode": _case("head64", "bf16", 6, "job", 16, 512, 128, 64, 1024, steps=1),
        "head64_job_paged": _case("head64", "bf16", 6, "job", 48, 384, 128, 64, 1200, steps=96, block=64),
        # One interactive request at the OPT-13B shape: its prompt, and a decode iteration, which streams 25.7 GB of weights.
        "opt13b_encode_1": _case("opt13b", "bf16", 20, "job", 1, 512, 0, 512, 512),
        "opt13b_decode_1": _case("opt13b", "bf16", 40, "decode", 1, 576, 0, 576, 576),
        # The decode batch a latency bound leaves, on a paged pool.
        "opt13b_decode_32_paged": _case("opt13b", "bf16", 40, "decode", 32, 576, 132, 80, 1280, block=64),
        # Ten of the forty layers (a quarter of the model, a pipeline stage's share with the LM head): the decode batch and
        # the encode batch of the throughput schedule.
        "opt13b_decode_256": _case("opt13b", "bf16", 10, "decode", 256, 576, 132, 80, 1280),
        "opt13b_encode_32": _case("opt13b", "bf16", 10, "job", 32, 512, 128, 64, 1024, steps=1),
        # The T5-11B shape: half of the layers, an encode batch of 16 with the first decode step.
        "t5_11b_encode_16": _case("t5_11b", "bf16", 12, "job", 16, 768, 192, 128, 1024, steps=1, enc_layers=12),
        # A third of a GPT-3-175B pipeline stage (hidden states in and out): an encode batch of 8, then decoding.
        "gpt3_share_job": _case("gpt3_share", "bf16", 4, "job", 8, 1024, 256, 128, 2048, steps=16),
    }
    return [dict(c, name=n) for n, c in named.items()]


def _log_int(rng, lo, hi):
    return int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))


def draw(rng):
    """One more case of the same ranges: batches and lengths over their logarithm, odd ones among them, with the depth
    cut where batch and length are large, so that none costs more than the largest listed case."""
    kind = rng.choice(["small_job", "small_t5", "small_encode", "head64_encode", "head64_job", "big_encode", "big_encode",
                       "big_decode", "big_decode", "big_decode", "t5_11b", "gpt3"])
    if kind == "small_job":
        n, m = _log_int(rng, 1, 32), _log_int(rng, 8, 200)
        return _case("tiny", rng.choice(["f32", "bf16"]), rng.randint(2, 4), "job", n, m, m // 4, 1, 2 * m, steps=rng.randint(8, 24))
    if kind == "small_t5":
        n, m = _log_int(rng, 2, 32), _log_int(rng, 16, 256)
        return _case("small_t5", rng.choice(["f32", "f32", "bf16"]), 2, "job", n, m, m // 4, 1, 2 * m, steps=rng.randint(8, 24))
    if kind == "small_encode":
        n, m = _log_int(rng, 4, 48), _log_int(rng, 64, 480)
        return _case("tiny", "f32", 2, "job", n, m, m // 4, 1, min(2 * m, 1000), steps=1)
    if kind == "head64_encode":
        n, m = _log_int(rng, 1, 24), _log_int(rng, 48, 900)
        return _case("head64", "bf16", rng.randint(2, 6), "job", n, m, m // 4, 1, min(2 * m, 1400), steps=1)
    if kind == "head64_job":
        n, m = _log_int(rng, 1, 96), _log_int(rng, 48, 700)
        return _case("head64", "bf16", rng.randint(2, 6), "job", n, m, m // 4, 1, min(2 * m, 1200), steps=rng.randint(32, 96),
                     block=rng.choice([0, 16, 64, 256]))
    if kind == "big_encode":
        n, m = _log_int(rng, 1, 32), _log_int(rng, 96, 900)
        layers = max(2, min(10, 160000 // (n * m)))
        return _case("opt13b", "bf16", layers, "job", n, m, m // 4, 1, min(2 * m, 1024), steps=rng.randint(0, 1))
    if kind == "big_decode":
        n, m = _log_int(rng, 1, 280), _log_int(rng, 64, 1000)
        layers = max(2, min(40, 1400000 // (n * m), 3200000 // (n * (m + 640))))
        return _case("opt13b", "bf16", layers, "decode", n, m, m // 4, 1, min(2 * m, 1280), block=rng.choice([0, 0, 64]))
    if kind == "t5_11b":
        m = _log_int(rng, 96, 900)
        n = _log_int(rng, 1, 48)
        if rng.random() < 0.5:
            layers = max(1, min(8, 110000 // (n * m)))
            return _case("t5_11b", "bf16", layers, "job", n, m, m // 4, 1, min(2 * m, 1024), steps=1, enc_layers=layers)
        return _case("t5_11b", "bf16", max(4, min(24, 400000 // (n * m))), "decode", n, m, m // 4, 1, min(2 * m, 1024),
                     enc_layers=2)
    n, m = _log_int(rng, 1, 12), _log_int(rng, 128, 1500)
    layers = max(1, min(4, 32000 // (n * m)))
    return _case("gpt3_share", "bf16", layers, "job", n, m, m // 4, 1, min(2 * m, 2048), steps=rng.randint(4, 16))


def _lengths(rng, case):
    """Input lengths of the case's distribution, nudged by a position here and there until they sum to batch * mean: a
    case has the same amount of work, and outputs of the same shape, for every seed."""
    n, lo, hi = case["batch"], case["lo"], case["hi"]
    lens = wl.clipped_normal_lengths(rng, n, case["mean"], case["std"], lo, hi)
    while (off := n * case["mean"] - int(lens.sum())) != 0:
        free = np.nonzero(lens < hi if off > 0 else lens > lo)[0]
        lens[rng.permutation(free)[:abs(off)]] += 1 if off > 0 else -1
    return lens


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    shape = s.shape = _shape(case)
    rng = np.random.default_rng(seed)
    n = case["batch"]
    s.enc_dec = shape.arch == wl.ARCH_ENC_DEC
    s.embed = bool(shape.has_embed)
    s.ids = np.arange(n, dtype=np.int32)
    s.lens = _lengths(rng, case)
    total = int(s.lens.sum())
    # decode: room to grow, up to the end of a learned position table
    s.room = 640 if case["phase"] == "decode" else case["steps"] + 1
    s.reserve = np.full(n, s.room, dtype=np.int32) if s.enc_dec else np.minimum(s.lens + s.room, shape.max_pos or 1 << 20)
    s.tokens = wl.random_tokens(rng, total, shape.vocab) if s.embed else None
    s.fed = rng.integers(0, max(shape.vocab, 1), size=(max(s.room, 1), n)).astype(np.int32)
    weights = wl.make_weights(shape, seed, device=DEV)
    s.hidden = None
    if not s.embed:
        s.hidden = (wl.random_hidden(seed + 1, total, shape.d_model, shape.dtype, DEV),
                    wl.random_hidden(seed + 2, n, shape.d_model, shape.dtype, DEV))
    kv_layers = shape.n_dec_layers if s.enc_dec else shape.n_layers
    per_position = kv_layers * 2 * shape.inner * (4 if shape.dtype == wl.DTYPE_F32 else 2)
    block = case["block"] or 8
    positions = int((-(-s.reserve // block) * block).sum()) + (int((-(-s.lens // 8) * 8).sum()) if s.enc_dec else 0)
    # a decode batch was encoded 32 prompts at a time
    s.chunk = n if case["phase"] != "decode" else min(n, 32)
    most = max(int(s.lens[i:i + s.chunk].sum()) for i in range(0, n, s.chunk))
    cfg = exe.config_from_shape(shape, kv_pool_bytes=positions * per_position, max_seqs=n, max_batch_tokens=most,
                                max_batch_seqs=n, kv_block_size=case["block"])
    torch.cuda.synchronize()
    torch.cuda.empty_cache()            # the generator's float temporaries go back to the device
    s.stream = torch.cuda.Stream()
    s.model = exe.Model(cfg, weights, stream=s.stream)
    dt = torch.float32 if shape.dtype == wl.DTYPE_F32 else torch.bfloat16
    calls = max(case["steps"], 1)
    if s.embed:
        s.step_out = torch.zeros((calls, n, shape.vocab), dtype=torch.float32, device=DEV)
        s.first_out = torch.zeros((total, shape.d_model), dtype=dt, device=DEV) if s.enc_dec else \
            torch.zeros((n, shape.vocab), dtype=torch.float32, device=DEV)
    else:
        s.step_out = torch.zeros((calls, n, shape.d_model), dtype=dt, device=DEV)
        s.first_out = torch.zeros((total, shape.d_model), dtype=dt, device=DEV)
    torch.cuda.synchronize()
    s.done = 0
    if case["phase"] == "decode":
        _admit(s)
    return s


def _admit(s):
    """Encodes the whole batch, `chunk` prompts at a time (a live batch's outputs of that are not asked for)."""
    off = np.concatenate([[0], np.cumsum(s.lens)])
    live = s.case["phase"] == "decode"
    for b in range(0, len(s.ids), s.chunk):
        e = min(len(s.ids), b + s.chunk)
        s.model.encode(s.ids[b:e], s.lens[b:e], s.tokens[off[b]:off[e]] if s.embed else None, reserve_lengths=s.reserve[b:e],
                       hidden_in=None if s.embed else s.hidden[0][off[b]:off[e]], want_tokens=s.embed and not s.enc_dec,
                       out_device=None if live else s.first_out)
    s.done = 0


def _step(s, out):
    before = 0 if s.enc_dec else s.lens
    kv = np.broadcast_to(np.asarray(before + s.done + 1, dtype=np.int32), s.lens.shape)
    s.model.decode_step(s.ids, s.fed[s.done] if s.embed else None, kv, hidden_in=None if s.embed else s.hidden[1],
                        want_tokens=s.embed, out_device=out)
    s.done += 1


def run(state):
    s = state
    if s.case["phase"] == "decode":
        # the shortest room any sequence has (a learned position table may end before the reservation does)
        if s.done >= min(s.room, int((s.reserve - (0 if s.enc_dec else s.lens)).min())):
            s.model.seq_release(s.ids)
            _admit(s)
        _step(s, s.step_out[0])
        return s.step_out
    _admit(s)
    for t in range(s.case["steps"]):
        _step(s, s.step_out[t])
    s.model.seq_release(s.ids)
    return [s.first_out, s.step_out] if s.case["steps"] else s.first_out


def work(case):
    """Per call: every weight it uses read once, the inputs' embedding or hidden rows, the cached keys and values that it
    reads or writes, the outputs; the multiply-adds of the projections and of attention."""
    sh = _shape(case)
    e = 4 if sh.dtype == wl.DTYPE_F32 else 2
    n, d, inner, f, V = case["batch"], sh.d_model, sh.inner, sh.d_ff, sh.vocab if sh.has_lm_head else 0
    T = n * case["mean"]
    sq = n * (case["mean"] ** 2 + case["std"] ** 2)
    enc_dec = sh.arch == wl.ARCH_ENC_DEC
    ffn, attn = 2 * d * f, 4 * d * inner
    bytes_, flops = 0.0, 0.0

    def step(ctx):
        """one decode iteration at a mean of ctx self-attention positions"""
        L = sh.n_dec_layers if enc_dec else sh.n_layers
        w = L * (ffn + attn + (2 * d * inner if enc_dec else 0)) + V * d
        kv = L * 2 * inner * n * (ctx + (case["mean"] if enc_dec else 0))
        return w * e + kv * e + L * 2 * inner * n * e + n * (V * 4 if V else 2 * d * e), 2.0 * n * w + 2.0 * kv

    if case["phase"] != "decode":
        w = sh.n_layers * (ffn + attn)
        bytes_ += w * e + T * d * e
        flops += 2.0 * T * w + sh.n_layers * (4.0 * inner * sq if enc_dec else 2.0 * inner * sq)
        if enc_dec:                     # cross keys and values of every decoder layer, and the encoder output
            wx = sh.n_dec_layers * 2 * d * inner
            bytes_ += wx * e + sh.n_dec_layers * 2 * inner * T * e + T * d * e
            flops += 2.0 * T * wx
        else:                           # cached keys and values; logits of the last positions, or hidden states
            bytes_ += sh.n_layers * 2 * inner * T * e + (V * d * e + n * V * 4 if V else T * d * e)
            flops += 2.0 * n * V * d
    for t in range(case["steps"] if case["phase"] == "job" else 1):
        b, fl = step((0 if enc_dec else case["mean"]) + t + 1)
        bytes_ += b
        flops += fl
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """Four times what was measured.  Float: against the same computation in 64 bits, rel 8e-7 and max 3.5e-6 on the small
    jobs.  bf16: against the same calls with every product's sums in another order (other tile shapes and no split-K), rel
    0.003 to 0.005 and max 0.015 to 0.025 over the listed cases."""
    if case["dtype"] == "f32":
        return {"rel": 3.2e-6, "max": 1.4e-5}
    return {"rel": 2e-2, "max": 0.1}
