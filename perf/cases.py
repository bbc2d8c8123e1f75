"""Performance cases of the branch-batched denoising path: block steps, full-sequence forwards and a whole decode,
through the package's public calls, over the shapes of `workload/configs.py` and generic sizes around them.

A case names a call sequence (`kind`), a model shape with its depth, and the requests it serves:

  step     denoise_step at a frozen state in the middle of a decode (one block forward of every listed request)
  refresh  refresh(BB_PERIODIC) of the listed requests and the block step that follows it (every R-th step of a decode)
  init     request_open, refresh(BB_INIT), request_close (a new request's first forward)
  decode   request_open, generate, get_tokens, request_close (a request from prompt to tokens)

Weights, prompts, decoded tokens and windows are made from the seed on the GPU or in the host's generator.  A large
model's depth is reduced where three states of full depth would not fit one card: the layers are alike, so the work per
layer and its kernels stay what they are at full depth.
"""
import numpy as np
import torch

from paper_2605_29233_amd import BB_INIT, BB_PERIODIC, BlockBatch, Limits
from workload import workload, weight_specs
from workload.configs import DREAM, LLADA, TINY, DecodeParams, scaled

_MODELS = {"tiny": TINY, "llada": LLADA, "dream": DREAM}
_DEVICE = "cuda:0"


def _case(name, kind, model, layers, prompts, gen, blocks, masked=0.6, refresh_interval=8):
    return {"name": name, "kind": kind, "model": model, "layers": layers, "prompts": ",".join(map(str, prompts)), "gen": gen,
            "blocks": ",".join(map(str, blocks)), "masked": masked, "refresh_interval": refresh_interval}


def _of(name, kind, layers=None, case_name=None, **kw):
    """A case of one of the named workloads' own shapes."""
    w = workload(name)
    model = {m.name: k for k, m in _MODELS.items()}[w.model.name]
    return _case(case_name or f"{name}_{kind}", kind, model, layers or w.model.n_layers, w.prompt_lens, w.gen_len, w.block_sizes,
                 refresh_interval=w.decode.refresh_interval, **kw)


def listed():
    return [
        # the smallest call: 56 rows of a two-layer model, where latency and the number of launches count
        _of("tiny", "step"),
        # a whole small request: initial forward, steps with commit / merge / sync, refreshes, tokens back on the host
        _of("tiny", "decode"),
        # one branch, block 32: plain cached block decoding of a single stream, weights read for 32 rows
        _of("llada_b32", "step"),
        # the headline workload: four branches, 120 rows, every weight streamed once per step
        _of("llada", "step"),
        # its periodic refresh (3072 rows) with the step behind it
        _of("llada", "refresh"),
        # a new request arriving: 768 rows, logits for all 256 generation positions
        _of("llada", "init"),
        # grouped-query model with biases and a longer row
        _of("dream", "step"),
        # the same model with a ragged prompt and generation length: no row count is a multiple of a tile
        _case("dream_ragged_refresh", "refresh", "dream", 28, (1013,), 389, (12, 32, 50)),
        # six branches with block sizes 4..128 (252 rows), windows partly decoded
        _of("llada_paper6", "step", layers=16),
        # many users at once: 16 requests x 4 branches, 1920 rows, ragged prompts
        _of("llada_x16", "step", layers=16),
        # long context: 240 rows against 5120 cached tokens per branch
        _of("llada_long", "step", layers=16),
        # its refresh: 4 x 5120 rows, attention over the whole row
        _of("llada_long", "refresh", layers=8),
    ]


def _ints(text):
    return [int(x) for x in text.split(",")]


def _sizes(case):
    """(model shape, prompt lengths, generation length, block sizes clipped to it)."""
    model = scaled(_MODELS[case["model"]], n_layers=case["layers"])
    gen = case["gen"]
    return model, _ints(case["prompts"]), gen, [min(b, gen) for b in _ints(case["blocks"])]


def _param_counts(m):
    """(parameters of one layer's matrices, of its key and value projections, of the LM head)."""
    nq, nkv = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    return (2 * nq + 2 * nkv + 3 * m.d_ffn) * m.d_model, 2 * nkv * m.d_model, m.vocab * m.d_model


def _cache_bytes(case):
    """Bytes of the largest buffers of a state: weights, K,V rows, activations of a full pass."""
    m, prompts, gen, blocks = _sizes(case)
    layer, _, lm = _param_counts(m)
    L = max(prompts) + gen
    kv = 8 * m.n_layers * len(prompts) * (len(blocks) + 1) * (L + 63) * m.n_kv_heads * m.head_dim
    rows = max(len(blocks) * L, len(prompts) * sum(blocks))
    lm_rows = max(gen, len(prompts) * sum(blocks))
    return 4 * m.n_layers * layer + 6 * lm + kv + rows * 4 * (6 * m.d_model + 6 * m.d_ffn) + 4 * lm_rows * m.vocab


def work(case):
    m, prompts, gen, blocks = _sizes(case)
    layer, kv_proj, lm = _param_counts(m)
    qd, kvd, nb = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim, len(blocks)
    Ls = [p + gen for p in prompts]

    def step(share=case["masked"]):
        rows = len(prompts) * sum(blocks)
        lm_rows = share * rows
        flops = 2.0 * rows * layer * m.n_layers + sum(4.0 * sum(blocks) * L * qd for L in Ls) * m.n_layers + 2.0 * lm_rows * lm
        bytes_ = 2.0 * (layer * m.n_layers + lm) + sum(2.0 * 2 * kvd * L * nb for L in Ls) * m.n_layers + 4.0 * lm_rows * m.vocab
        return np.array([bytes_, flops])

    def full(rows_per_request, lm_rows):
        """A pass over whole rows; without an LM head it ends with the last layer's keys and values."""
        rows = sum(r for r, _ in rows_per_request)
        depth = m.n_layers if lm_rows else m.n_layers - 1
        flops = 2.0 * rows * layer * depth + sum(4.0 * r * L * qd for r, L in rows_per_request) * depth
        flops += 2.0 * lm_rows * lm if lm_rows else 2.0 * rows * kv_proj
        bytes_ = 2.0 * (layer * depth + (lm if lm_rows else kv_proj)) + 2.0 * 2 * kvd * rows * m.n_layers + 4.0 * lm_rows * m.vocab
        return np.array([bytes_, flops])

    if case["kind"] == "step":
        total = step()
    elif case["kind"] == "refresh":
        total = full([(nb * L, L) for L in Ls], 0) + step()
    elif case["kind"] == "init":
        total = full([(L, L) for L in Ls], gen)
    else:                       # decode: at least one block forward per window of the widest branch, a refresh every R of them
        forwards = -(-gen // max(blocks))
        total = full([(L, L) for L in Ls], gen) + forwards * step() + forwards // case["refresh_interval"] * full([(nb * L, L) for L in Ls], 0)
    return {"bytes": float(total[0]), "flops": float(total[1])}


def tolerance(case):
    """Four times what the same passes differ by when the layer GEMMs take two bf16 terms per activation instead of
    fp16 + fp8 (another format of the same precision, BlockBatch.wide_format): the confidences differ most, by 4.1e-4 of
    their norm and 1.5e-3 of a value at 16 to 32 layers (logits 1.4e-4 and 1.4e-3), by 5.6e-5 and 1.0e-4 in the two-layer
    model.  Two logits of a row within that of each other may change the row's token: 2 of 1152 rows did."""
    if case["kind"] == "decode":
        return {"rel": 2.5e-4, "max": 5e-4, "differ": 0.0}
    if case["model"] == "tiny":
        return {"rel": 2.5e-4, "max": 5e-4, "differ": 0.01}
    return {"rel": 1.6e-3, "max": 6e-3, "differ": 0.01}


def draw(rng):
    """Another case of these ranges: sizes spread over their logarithm, odd ones among them, at most the cost of the
    largest listed case, and a state that fits the card three times over."""
    top = max(work(c)["flops"] for c in listed())

    def log_int(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    while True:
        model = rng.choice(("tiny", "llada", "llada", "dream"))
        kind = rng.choice(("step", "step", "step", "refresh", "init") + (("decode",) if model == "tiny" else ()))
        small = model == "tiny"
        layers = 2 if small else log_int(4, _MODELS[model].n_layers)
        requests = log_int(1, 16) if kind == "step" else 1
        prompts = [log_int(16, 192 if small else 4096) for _ in range(requests)]
        gen = log_int(24, 128 if small else 1024)
        blocks = sorted({log_int(4, 32 if small else 128) for _ in range(rng.randint(1, 6))})
        case = _case("", kind, model, layers, prompts, gen, blocks, masked=round(rng.uniform(0.3, 1.0), 2), refresh_interval=rng.choice((4, 8, 16)))
        del case["name"]
        if work(case)["flops"] <= top and _cache_bytes(case) <= 80e9:
            return case


class _Window:
    """One branch of set_state: its window and the mean confidence of its latest decode."""

    def __init__(self, start, end):
        self.start, self.end, self.done, self.mean_conf = start, end, 0, 0.5


def _weights(model, seed):
    """The tensors of `workload.weight_specs`, drawn on the GPU: matrices N(0, std), norm gains around 1."""
    g = torch.Generator(device=_DEVICE)
    g.manual_seed(seed)
    for name, shape, kind in weight_specs(model):
        t = torch.empty(shape, dtype=torch.bfloat16, device=_DEVICE)
        if kind == "ones":
            yield name, t.normal_(1.0, 0.05, generator=g)
        else:
            yield name, t.normal_(0.0, model.lm_head_std if kind == "lm" else model.w_std, generator=g)


def _mid_decode(rng, model, prompt, gen, blocks, masked):
    """Rows and windows of a request in the middle of its decode: every branch has decoded the windows before its own
    (the branches agree on the tokens), and a share of its own window."""
    L_p, L = len(prompt), len(prompt) + gen
    truth = rng.integers(0, model.vocab - 1, gen, dtype=np.int32)
    X = np.full((len(blocks), L), model.mask_id, dtype=np.int32)
    windows, n_masked = [], 0
    for k, b in enumerate(blocks):
        X[k, :L_p] = prompt
        first = int(rng.integers(0, max(1, (3 * gen // 4) // b)))      # (a whole window: the row count is the same for every seed)
        start = L_p + first * b
        end = start + b
        X[k, L_p:end] = truth[:end - L_p]
        n = max(1, round(masked * b))
        X[k, start + rng.permutation(b)[:n]] = model.mask_id
        n_masked += n
        windows.append(_Window(start, end))
    return X, windows, n_masked


class _State:
    pass


def prepare(case, seed):
    model, prompt_lens, gen, blocks = _sizes(case)
    rng = np.random.default_rng(seed)
    L = max(prompt_lens) + gen
    small = case["model"] == "tiny"
    decode = DecodeParams(refresh_interval=case["refresh_interval"], leader_rule=1 if small else 0)
    s = _State()
    s.kind, s.gen, s.blocks = case["kind"], gen, blocks
    s.bb = BlockBatch(model, decode, Limits(len(prompt_lens), len(blocks), L, gen, len(prompt_lens) * sum(blocks)), device=_DEVICE)
    s.bb.load_weights(_weights(model, seed))
    s.bb.keep_logits(s.kind != "decode")           # the rows' logits are results here, beside token and confidence
    prompts = [rng.integers(0, model.vocab - 1, n, dtype=np.int32) for n in prompt_lens]
    s.prompt = prompts[0]
    s.ids = []
    if s.kind in ("step", "refresh"):
        rows = 0
        s.ids = [s.bb.request_open(p, gen, blocks) for p in prompts]
        for rid, p in zip(s.ids, prompts):
            s.bb.refresh([rid], BB_INIT)
            X, windows, n = _mid_decode(rng, model, p, gen, blocks, case["masked"])
            s.bb.set_state(rid, X, windows)
            rows += n
        s.bb.refresh(s.ids, BB_PERIODIC)
    else:
        rows = gen
    if s.kind != "decode":
        s.view = _device_view(s.bb, rows, model.vocab)
    s.bb.synchronize()
    torch.cuda.empty_cache()                       # what making the weights took
    return s


def _device_view(bb, rows, vocab):
    """The results of the latest forward (bb_step_view) as tensors over the workspace."""
    raw = bb.latest_view()._raw

    def at(ptr, n, dtype):
        off = ptr - bb._ws.data_ptr()
        return bb._ws[off:off + n * 4].view(dtype)

    return {"argmax": at(raw.argmax_dev, rows, torch.int32), "conf": at(raw.conf_dev, rows, torch.float32),
            "lse": at(raw.lse_dev, rows, torch.float32), "logits": at(raw.logits_dev, rows * vocab, torch.float32).view(rows, vocab)}


def run(s):
    bb = s.bb
    if s.kind == "decode":
        rid = bb.request_open(s.prompt, s.gen, s.blocks)
        st = bb.generate([rid])[0]
        X = bb.get_tokens(rid)
        bb.request_close(rid)
        branches = list(st.branch)[:st.n_branches]
        return {"tokens": X, "winner": st.winner, "forwards": np.array([st.nfe_init, st.nfe_block, st.nfe_refresh]),
                "merged": np.array([b.tokens_merged for b in branches]), "mean_conf": np.array([b.mean_conf for b in branches])}
    if s.kind == "init":
        rid = bb.request_open(s.prompt, s.gen, s.blocks)
        bb.refresh([rid], BB_INIT)
        bb.request_close(rid)
        return s.view
    if s.kind == "refresh":
        bb.refresh(s.ids, BB_PERIODIC)
    bb.denoise_step(s.ids, want_view=False)
    return s.view
