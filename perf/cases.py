"""The cases on which this library's speed is measured: what its users have it do, through the public calls.

A training step is a forward and a backward call, a prefill a forward call alone, a decode step one
query per head against a cache.  Sizes are those of `workloads.CONFIGS`, of the benchmark's sweeps
and of the tests.  Inputs are drawn on the GPU by the recipes of `workloads.py`:

* "gaussian": Q, K ~ N(0, sigma^2), V, dO ~ N(0, 1), independent rows;
* "block":    the 64 query rows of a tile share most of their direction, so that whole 64 x 64 blocks
              of the attention matrix are empty;
* "planted":  every query tile attends to 32 earlier keys (a long context with high block sparsity).

sigma steers how many keys a row attends to: about 26 of 16384 at sigma = 1, 2 at sigma = 4 (d = 128).
"""
import math

import torch

import paper_2604_15180_amd as ea

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _train(name, B, H, N, d, alpha, sigma, dtype="bf16", causal=True, inputs="gaussian", lists=True):
    # lists: the backward is handed the forward's workspace (the benchmark's training step); else it
    # gets the mask alone (a caller that reuses the workspace between layers)
    return dict(name=name, kind="train", B=B, H=H, N=N, d=d, dtype=dtype, alpha=alpha, causal=causal,
                inputs=inputs, sigma=sigma, lists=lists)


def listed():
    return [
        # the smallest training step, fp32 and without a mask: launches and host work count
        _train("train_f32_256", 1, 2, 256, 64, 1.5, 1.0, dtype="f32", causal=False, lists=False),
        # a small model's step at a sequence length that fills no power of two
        _train("train_bf16_1088", 2, 8, 1088, 64, 1.5, 1.5),
        # an ordinary pre-training step: 64 heads of 4096 tokens, moderate sparsity
        _train("train_bf16_4k", 4, 16, 4096, 64, 1.5, 1.5),
        # alpha away from the closed forms (power functions in every kernel)
        _train("train_bf16_8k_a125", 2, 16, 8192, 64, 1.25, 2.0),
        # sparsemax, the backward without the forward's lists
        _train("train_bf16_8k_a2", 2, 16, 8192, 64, 2.0, 2.0, lists=False),
        # the headline sweep at its dense end, at a sparse point, and with block-structured sparsity
        _train("train_bf16_16k_s1", 2, 16, 16384, 128, 1.5, 1.0),
        _train("train_bf16_16k_s3", 2, 16, 16384, 128, 1.5, 3.0),
        _train("train_bf16_16k_block", 2, 16, 16384, 128, 1.5, 2.0, inputs="block"),
        # long context: few heads, planted keys, 96 % of the blocks empty
        _train("train_bf16_64k", 1, 8, 65536, 128, 1.5, 3.0, inputs="planted"),
        # a prompt of odd length run through the forward alone
        dict(name="prefill_bf16_3136", kind="prefill", B=1, H=32, N=3136, d=128, dtype="bf16", alpha=1.5,
             causal=True, inputs="gaussian", sigma=2.0),
        # one generated token: at the start of a conversation, and against a full cache
        dict(name="decode_bf16_1000", kind="decode", B=1, H=32, N=1000, d=128, dtype="bf16", alpha=1.5, sigma=3.0),
        dict(name="decode_bf16_128k", kind="decode", B=1, H=32, N=131072, d=128, dtype="bf16", alpha=1.5, sigma=3.0),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choices(("train", "prefill", "decode"), (6, 2, 2))[0]
    d = rng.choice((64, 128))
    dtype = rng.choices(("bf16", "f32"), (7, 1))[0]
    alpha = rng.choice((1.25, 1.5, 1.5, 1.5, 1.75, 2.0))
    sigma = round(rng.uniform(1.0, 4.0), 2)
    B = rng.choice((1, 2, 4))
    if kind == "decode":
        N = int(_log_uniform(rng, 500, 131072))
        most = 32 * 131072 * 128 * 2 // (N * d * (4 if dtype == "f32" else 2))      # the listed cache's bytes
        H = max(1, min(rng.choice((4, 8, 12, 16, 32)), most // B))
        return dict(kind=kind, B=B if B * H <= most else 1, H=H, N=N, d=d, dtype=dtype, alpha=alpha, sigma=sigma)
    causal = rng.random() < 0.85
    N = 64 * max(1, int(_log_uniform(rng, 3, 1024)))
    if dtype == "f32":
        N = min(N, 64 * rng.randint(16, 40))
        sigma = min(sigma, 2.0)
    inputs = rng.choices(("gaussian", "block", "planted"), (3, 1, 1))[0] if dtype == "bf16" and N >= 1024 else "gaussian"
    # no more scores than the listed step at 16384 tokens; without a mask twice as many are visible,
    # with power functions or in fp32 each is several times the work
    weight = (1 if causal else 2) * (1 if alpha in (1.5, 2.0) else 4) * (8 if dtype == "f32" else 1)
    most = 32 * 16384.0 * 16384.0 / (N * float(N) * weight)
    heads = max(1, min(int(most), rng.choice((4, 8, 12, 16, 32, 64))))
    B = B if heads % B == 0 else 1
    case = dict(kind=kind, B=B, H=heads // B, N=N, d=d, dtype=dtype, alpha=alpha, causal=causal, inputs=inputs, sigma=sigma)
    if kind == "train":
        case["lists"] = rng.random() < 0.7
    if most < 1:
        case["alpha"], case["causal"] = 1.5, True       # one head of the longest sequences, in its usual form
    return case


def _inputs(case, gen):
    B, H, N, d, sigma = case["B"], case["H"], case["N"], case["d"], case["sigma"]
    normal = lambda *shape: torch.randn(*shape, generator=gen, device=gen.device)  # noqa: E731
    q, k = normal(B, H, N, d), normal(B, H, N, d)
    if case["inputs"] == "block":
        shared = normal(B, H, N // 64, 1, d)
        q = (math.sqrt(0.98) * shared + math.sqrt(0.02) * q.view(B, H, N // 64, 64, d)).reshape(B, H, N, d)
    q, k = q * sigma, k * sigma
    if case["inputs"] == "planted":
        T = N // 64
        strength = math.sqrt(60.0 * math.sqrt(d))
        dirs = normal(B, H, T, d)
        dirs = dirs / dirs.norm(dim=-1, keepdim=True) * strength
        dirs[:, :, 0] = 0.0                               # tile 0 has no earlier keys
        q = (q.view(B, H, T, 64, d) + dirs.unsqueeze(3)).reshape(B, H, N, d)
        where = torch.rand(B, H, T, 32, generator=gen, device=gen.device)
        for i in range(1, T):
            pos = (where[:, :, i] * (64 * i)).long().clamp_(max=64 * i - 1)
            k.scatter_add_(2, pos.unsqueeze(-1).expand(B, H, 32, d), dirs[:, :, i].unsqueeze(2).expand(B, H, 32, d).contiguous())
    return q, k, normal(B, H, N, d)


def prepare(case, seed):
    gen = torch.Generator(device="cuda:0").manual_seed(int(seed))
    dtype, shape = DTYPES[case["dtype"]], (case["B"], case["H"], case["N"], case["d"])
    if case["kind"] == "decode":
        B, H, N, d = shape
        q = torch.randn(B, H, d, generator=gen, device=gen.device) * case["sigma"]
        k = torch.randn(B, H, N, d, generator=gen, device=gen.device) * case["sigma"]
        v = torch.randn(B, H, N, d, generator=gen, device=gen.device)
        ws = torch.empty(ea.entmax_attn_decode_workspace_bytes(*shape, dtype), dtype=torch.uint8, device=gen.device)
        return dict(case=case, q=q.to(dtype), K=k.to(dtype), V=v.to(dtype), ws=ws)
    q, k, v = _inputs(case, gen)
    state = dict(case=case, Q=q.to(dtype), K=k.to(dtype), V=v.to(dtype))
    bytes_of = lambda is_bwd: ea.entmax_attn_workspace_bytes(*shape, dtype, case["causal"], is_bwd)  # noqa: E731
    state["ws_f"] = torch.empty(bytes_of(False), dtype=torch.uint8, device=gen.device)
    if case["kind"] == "train":
        state["dO"] = torch.randn(*shape, generator=gen, device=gen.device).to(dtype)
        state["ws_b"] = torch.empty(bytes_of(True), dtype=torch.uint8, device=gen.device)
    return state


def run(state):
    case = state["case"]
    alpha = case["alpha"]
    if case["kind"] == "decode":
        O, tau, _, _ = ea.entmax_attn_decode(state["q"], state["K"], state["V"], alpha, workspace=state["ws"])
        return dict(O=O, tau=tau)
    Q, K, V, causal = state["Q"], state["K"], state["V"], case["causal"]
    O, tau, mask = ea.entmax_attn_fwd(Q, K, V, alpha, causal, workspace=state["ws_f"])
    if case["kind"] == "prefill":
        return dict(O=O, tau=tau, mask=mask)
    dQ, dK, dV = ea.entmax_attn_bwd(Q, K, V, O, state["dO"], tau, alpha, causal, block_mask=mask, workspace=state["ws_b"],
                                    fwd_workspace=state["ws_f"] if case["lists"] else None)
    return dict(O=O, tau=tau, mask=mask, dQ=dQ, dK=dK, dV=dV)


def work(case):
    BH, N, d = case["B"] * case["H"], case["N"], case["d"]
    size = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "decode":
        # the keys, and one product with each; the few rows of V that are attended to depend on the inputs
        return dict(bytes=BH * (N * d * size + d * size + d * 4 + 4), flops=2.0 * BH * N * d)
    # forward: every visible score once; what is done for the non-zero probabilities alone (a few
    # keys of thousands, depending on the inputs) is left out
    pairs = N * (N + 64) / 2 if case["causal"] else N * float(N)
    tensor = BH * N * d
    moved = 3 * tensor * size + tensor * 4 + BH * N * 4 + BH * (N // 64) * ((N // 64 + 31) // 32) * 4
    if case["kind"] == "train":
        moved += 4 * tensor * size + tensor * 4 + BH * N * 4 + 3 * tensor * 4
    return dict(bytes=moved, flops=2.0 * BH * pairs * d)


def tolerance(case):
    """About four times what one head of each kind of case differs from the same path in float64 torch.
    bf16: 2.1e-4 of O where P goes through the matrix cores as fp16 (2^-12 per element), 5e-5 of the
    gradients, where the refinement stops within 1e-4 of the threshold's root; largest single error
    1.8e-3.  fp32: 2.5e-6, largest 2.7e-5.  alpha = 1.75: U = P^(1/4) has an unbounded slope at the
    support's edge: 2.5e-5 in fp32 too, largest 2.7e-3.  alpha = 2: U is 0 or 1, and a key within the
    threshold's accuracy of the edge may be on either side of it - one entry of its row.  Decode
    sums in fp32 from a threshold known to 1e-4.  A mask word may differ for such keys as well."""
    if case["kind"] == "decode":
        return dict(rel=1e-4, max=1e-3)
    alpha, f32 = case["alpha"], case["dtype"] == "f32"
    rel = 1e-3 if not f32 else 1e-5 if alpha in (1.25, 1.5, 2.0) else 1e-4
    most = 0.9 if alpha == 2.0 else 1e-2 if alpha == 1.75 else 1.1e-4 if f32 else 8e-3
    return dict(rel=rel, max=most, differ=1e-3)
