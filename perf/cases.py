"""The workloads this framework's speed is judged by: the stage calls a co-located trainer and server makes.

Every case is one call (or one training task) through `binding.Stage` on one of the named stage configurations of
`synth_inputs.CONFIGS`, possibly with another number of blocks:

  train    stage_train_fwd + stage_train_bwd over `micro` micro-batches of batch x length tokens (the second one
           accumulates into the same gradients); outputs Y, dX of each and the parameter gradients
  decode   one stage_decode step of `batch` requests over a paged cache with the case's context lengths
  prefill  one stage_prefill of several prompt chunks, each behind `past` cached tokens
  step     one stage_step: decode rows and prompt chunks in one forward (what the batching server issues)
  update   one stage_optimizer_step (AdamW) over the stage's parameters

X, dY, weights and cache rows are Gaussian with the configurations' scales; pages are shuffled.
"""
import math

import torch

from paper_2507_21276_amd import binding as B
from paper_2507_21276_amd import synth_inputs as S

TINY, GPT, L7, L13 = "tiny_gpt_f32", "gpt2s_bf16", "llama7b_bf16", "llama13b_bf16"


def listed():
    return [
        # the smallest training task: the fp32 stage, 128 tokens; a chain of launches
        dict(name="tiny_train_f32", kind="train", model=TINY, layers=2, mma="f32", micro=1, batch=2, length=64),
        # one request decoding alone on a small stage: per-token latency
        dict(name="small_decode_1", kind="decode", model=GPT, layers=6, mma="f16", batch=1, ctx_lo=77, ctx_hi=77, lengths=0),
        # the small stage's ordinary decode batch, equal contexts
        dict(name="small_decode_32", kind="decode", model=GPT, layers=6, mma="f16", batch=32, ctx_lo=512, ctx_hi=512, lengths=0),
        # the small stage's ordinary micro-batch
        dict(name="small_train_4x1024", kind="train", model=GPT, layers=6, mma="f16", micro=1, batch=4, length=1024),
        # two short micro-batches of ragged length (query / reference pairs are rarely a power of two), bf16 operands
        dict(name="small_train_3x333", kind="train", model=GPT, layers=6, mma="bf16", micro=2, batch=3, length=333),
        # the model update that follows every training task
        dict(name="small_update", kind="update", model=GPT, layers=6, mma="f16"),
        # one request decoding alone on a large stage: every weight is read for one row
        dict(name="large_decode_1", kind="decode", model=L7, layers=8, mma="f16", batch=1, ctx_lo=1537, ctx_hi=1537, lengths=0),
        # the serving batch of the co-located mix: 64 requests of uneven length
        dict(name="large_decode_64", kind="decode", model=L7, layers=8, mma="f16", batch=64, ctx_lo=128, ctx_hi=2048, lengths=0),
        # prompt chunks as the server cuts them: one fresh, one continuing, one short rest
        dict(name="large_prefill_890", kind="prefill", model=L7, layers=8, mma="f16", chunks="512,301,77", past="0,512,1030"),
        # a hybrid mini-batch: running decodes and one admitted prompt, bf16 operands
        dict(name="large_step_48_200", kind="step", model=L7, layers=8, mma="bf16", batch=48, ctx_lo=64, ctx_hi=3000, lengths=1,
             chunks="200", past="0"),
        # the largest training task
        dict(name="large_train_2x2048", kind="train", model=L7, layers=8, mma="f16", micro=1, batch=2, length=2048),
        # the widest stage's decode batch with long-tailed contexts
        dict(name="wide_decode_128", kind="decode", model=L13, layers=4, mma="f16", batch=128, ctx_lo=64, ctx_hi=4096, lengths=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case of the same ranges; none needs more than the largest listed one."""
    kind = rng.choice(["train", "train", "decode", "decode", "prefill", "step", "update"])
    model = rng.choice([GPT, GPT, GPT, L7, L7, L7, L13] + ([TINY] if kind != "update" else []))
    depth = {TINY: 2, GPT: 12, L7: 8, L13: 4}[model]
    case = dict(kind=kind, model=model, layers=rng.randint(1, depth),
                mma="f32" if model == TINY else rng.choice(["f16", "f16", "bf16"]))
    if kind == "train":
        tokens = _log_int(rng, 16, 512) if model == TINY else _log_int(rng, 100, 4096)
        micro = rng.choice([1, 1, 2])
        batch = rng.randint(1, max(1, min(16, tokens // micro // 64)))
        case.update(micro=micro, batch=batch, length=max(8, tokens // micro // batch))
    if kind in ("decode", "step"):
        hi = 96 if model == TINY else _log_int(rng, 64, 1024) if model == GPT else _log_int(rng, 128, 4096)
        case.update(batch=_log_int(rng, 1, 8 if model == TINY else 128), ctx_lo=_log_int(rng, 16, hi), ctx_hi=hi,
                    lengths=rng.randint(1, 1 << 20))
    if kind in ("prefill", "step"):
        n = rng.randint(1, 6 if kind == "prefill" else 2)
        most = 64 if model == TINY else 512
        case["chunks"] = ",".join(str(_log_int(rng, 8, most)) for _ in range(n))
        case["past"] = ",".join(str(rng.choice([0, 0, rng.randint(1, most), rng.randint(1, most) * 2])) for _ in range(n))
    return case


def _config(case):
    return S.scaled(S.CONFIGS[case["model"]], n_layers=case["layers"])


def _numbers(text):
    return [int(v) for v in text.split(",")]


def _contexts(case):
    """Context length of each decoding request: fixed by the case (the work of a pass is known before it runs)."""
    lo, hi, n = case["ctx_lo"], case["ctx_hi"], case["batch"]
    return [int(v) for v in S.uniform_ints(case["lengths"], "contexts", n, lo, hi)]


def _requests(case):
    """(cached tokens, new tokens) of every request of a serving call, decode rows first."""
    old, new = [], []
    if case["kind"] in ("decode", "step"):
        old += _contexts(case)
        new += [1] * case["batch"]
    if case["kind"] in ("prefill", "step"):
        old += _numbers(case["past"])
        new += _numbers(case["chunks"])
    return old, new


def _stage(cfg, case, seed):
    stage = B.Stage(cfg, io_dtype=cfg["dtype"], mma_dtype=case["mma"])
    params = S.make_params_torch(cfg, seed)
    stage.ls_bind_params(params)
    return stage, params


def _cache(stage, cfg, case, seed):
    old, new = _requests(case)
    table, n_pages = S.page_tables(old, new, cfg["page_size"], seed)
    kv = B.KV(stage, n_pages, table, old)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 2 + 1)
    kv.k_pool.normal_(generator=g)
    kv.v_pool.normal_(generator=g)
    return kv


def prepare(case, seed):
    cfg = _config(case)
    stage, params = _stage(cfg, case, seed)
    io, d = stage.io_torch, cfg["d_model"]
    st = dict(kind=case["kind"], stage=stage, params=params)
    if case["kind"] == "train":
        n, b, length = case["micro"], case["batch"], case["length"]
        dy_std = 1.0 if cfg["block"] == "gpt" else 1e-2
        st.update(batch=b, length=length,
                  X=[S.normal_torch(seed, "X%d" % i, (b, length, d), 1.0, dtype=io) for i in range(n)],
                  dY=[S.normal_torch(seed, "dY%d" % i, (b, length, d), dy_std, dtype=io) for i in range(n)],
                  Y=[torch.empty(b, length, d, dtype=io, device="cuda") for _ in range(n)],
                  dX=[torch.empty(b, length, d, dtype=io, device="cuda") for _ in range(n)],
                  dParams=torch.empty(stage.ls_param_count(), dtype=torch.float32, device="cuda"),
                  saved=stage.new_saved(b, length), workspace=stage.new_workspace(b * length))
    elif case["kind"] == "update":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed * 2 + 1)
        n = stage.ls_param_count()
        new = lambda std: torch.empty(n, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=g)  # noqa: E731
        st.update(master=params.float(), m=new(1e-3), v=new(1e-3).square_(), dParams=new(1e-2), at=100)
    else:
        old, new = _requests(case)
        rows = sum(new)
        st.update(kv=_cache(stage, cfg, case, seed), batch=case.get("batch", 0),
                  chunks=_numbers(case["chunks"]) if "chunks" in case else [],
                  X=S.normal_torch(seed, "X", (rows, d), 1.0, dtype=io),
                  Y=torch.empty(rows, d, dtype=io, device="cuda"), workspace=stage.new_workspace(rows))
    return st


def run(st):
    stage, kind = st["stage"], st["kind"]
    if kind == "train":
        b, length = st["batch"], st["length"]
        for i, (x, dy, y, dx) in enumerate(zip(st["X"], st["dY"], st["Y"], st["dX"])):
            stage.stage_train_fwd(x, b, length, y, st["saved"], st["workspace"])
            stage.stage_train_bwd(dy, b, length, st["saved"], dx, st["dParams"], i > 0, st["workspace"])
        return dict(Y=st["Y"], dX=st["dX"], dParams=st["dParams"])
    if kind == "update":
        st["at"] += 1
        stage.stage_optimizer_step(st["params"], st["master"], st["m"], st["v"], st["dParams"], kind=B.LS_OPT_ADAMW,
                                   lr=1e-4, step=st["at"], weight_decay=0.01)
        return dict(params=st["params"], master=st["master"], m=st["m"], v=st["v"])
    kv = st["kv"]
    if kind == "decode":
        stage.stage_decode(st["X"], st["batch"], kv, st["Y"], st["workspace"])
    elif kind == "prefill":
        stage.stage_prefill(st["X"], st["chunks"], kv, st["Y"], st["workspace"])
    else:
        stage.stage_step(st["X"], st["batch"], st["chunks"], kv, st["Y"], st["workspace"])
    return dict(Y=st["Y"], k_pool=kv.k_pool, v_pool=kv.v_pool)  # the pools hold the new rows: updated state


def work(case):
    cfg = _config(case)
    d, n, layers = cfg["d_model"], S.param_count(cfg), cfg["n_layers"]
    size = 4 if cfg["dtype"] == "f32" else 2
    if case["kind"] == "update":
        # gradient, moments and master weights in; moments, master, stored and operand-format parameters out
        return dict(bytes=n * (16 + 12 + size + (2 if case["mma"] == "f16" else 0)), flops=0)
    if case["kind"] == "train":
        rows = case["micro"] * case["batch"] * case["length"]
        pairs = case["micro"] * case["batch"] * case["length"] * (case["length"] + 1) // 2
        return dict(bytes=n * (size + 4) + 4 * rows * d * size, flops=3 * (2.0 * n * rows + 4.0 * d * layers * pairs))
    old, new = _requests(case)
    rows = sum(new)
    cached = sum(o for o, _ in zip(old, new)) * 2 * d * layers * size
    pairs = sum(o * t + t * (t + 1) // 2 for o, t in zip(old, new))
    return dict(bytes=n * size + cached + rows * 2 * d * (size + size * layers), flops=2.0 * n * rows + 4.0 * d * layers * pairs)


def tolerance(case):
    """About four times the distance to the same path in float64 (Y, dX and the parameter gradients, measured on these
    configurations): the 16-bit storage of activations and results for the matrix-core modes, fp32 sums otherwise."""
    if case["kind"] == "update":
        return {"rel": 2e-5, "max": 1e-2}  # elementwise; a stored bf16 parameter may round the other way
    return {"f32": {"rel": 1.2e-6, "max": 2e-5}, "f16": {"rel": 8e-3, "max": 0.12}, "bf16": {"rel": 2e-2, "max": 0.5}}[case["mma"]]
