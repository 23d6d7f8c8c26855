"""Performance cases: calls of the MoE expert layer that a program serving or prefilling with it makes.

Every case is one call of `cq_moe_forward` (rotate, quantize, route, group, gate/up and down products on clustered
weights, combine) on a layer that lives on the GPU, for one of the model shapes that the repository's configurations
name.  A serving program calls it with 1..64 tokens per step, a prefill or chunked-prefill program with hundreds to
thousands; the layer's options are the activation bits (8 or 4), the online-Hadamard variant, block-wise centroid
tables and the 2-bit centroid budget.

  listed()               the cases that are always timed
  draw(rng)              one more case of the same ranges
  prepare(case, seed)    layer and tokens on the GPU
  run(state)             the call
  work(case)             bytes and operations it cannot do without
  tolerance(case)        how far a correct implementation of the same precision may be off
  exact(case, seed)      the same layer in float64, in plain torch
"""
import math

import torch

from paper_2604_10496_amd import binding, synth

# shape of a model's expert layer: the repository's own configurations
SHAPES = {"tiny": "tiny", "mixtral": "mixtral_decode", "dsv2lite": "dsv2lite", "qwen3": "qwen3_zipf"}
# the largest batch drawn for a variant: what its programs call it with, and nothing dearer than the largest listed
# case (block-wise tables cost a little more per token; the 2-bit format is meant for decode-sized batches; the tiny
# configuration stands for small calls)
MAX_TOKENS = {"plain": 4096, "had": 4096, "blockwise": 2048, "w2": 64}
BLOCK = 1024        # weights per table of the block-wise setting


def _case(model, variant, T, act_bits, name=None):
    c = {"model": model, "variant": variant, "T": T, "act_bits": act_bits}
    if name:
        c = {"name": name, **c}
    return c


def listed():
    return [
        # a small layer: launches and the host are what counts
        _case("tiny", "plain", 64, 8, "tiny_T64"),
        # one user's next token
        _case("mixtral", "plain", 1, 8, "mixtral_T1"),
        # a decode batch of 16: the configuration that the headline metric is quoted on
        _case("mixtral", "plain", 16, 8, "mixtral_T16"),
        # continuous batching with a ragged number of sequences, or a short chunk of prefill
        _case("mixtral", "plain", 77, 8, "mixtral_T77"),
        # a prompt of 512 tokens
        _case("mixtral", "plain", 512, 4, "mixtral_T512"),
        # prefill of a large batch
        _case("mixtral", "plain", 4096, 4, "mixtral_T4096"),
        # decode batch of 16 on many small experts with shared ones
        _case("dsv2lite", "plain", 16, 8, "dsv2lite_T16"),
        # a prompt on the same
        _case("dsv2lite", "plain", 512, 8, "dsv2lite_T512"),
        # prefill on many small experts whose popularity is skewed
        _case("qwen3", "plain", 2048, 4, "qwen3_T2048"),
        # prefill of the online-Hadamard variant, an odd number of tokens
        _case("mixtral", "had", 1001, 4, "mixtral_had_T1001"),
        # decode batch with one centroid table per 1024 weights
        _case("mixtral", "blockwise", 16, 8, "mixtral_blockwise_T16"),
        # decode batch with four centroids per row, two bits per weight
        _case("mixtral", "w2", 16, 8, "mixtral_w2_T16"),
    ]


def draw(rng):
    model, variant = rng.choice([("tiny", "plain"), ("mixtral", "plain"), ("mixtral", "plain"), ("mixtral", "plain"),
                                 ("dsv2lite", "plain"), ("dsv2lite", "plain"), ("qwen3", "plain"), ("qwen3", "plain"),
                                 ("mixtral", "had"), ("dsv2lite", "had"), ("qwen3", "had"),
                                 ("mixtral", "blockwise"), ("mixtral", "w2")])
    most = MAX_TOKENS[variant] if model != "tiny" else 512
    T = max(1, min(most, int(round(math.exp(rng.uniform(0.0, math.log(most + 0.5)))))))
    return _case(model, variant, T, rng.choice([4, 8]))


def _config(case):
    base = synth.CONFIGS[SHAPES[case["model"]]]
    over = {"T": case["T"], "act_bits": case["act_bits"], "outlier_channels": ()}
    if case["variant"] == "had":
        over.update(h_bits=case["act_bits"], r_hadamard=True)
    elif case["variant"] == "blockwise":
        over.update(group_k=BLOCK)
    elif case["variant"] == "w2":
        over.update(index_bits=2)
    return synth.small_variant(base, **over)


# ------------------------------------------------------------------------------------------------
# inputs (drawn on the GPU; the distributions of synth.py)
# ------------------------------------------------------------------------------------------------
def _centroids(gen, G, N, tables, budget):
    """[G, N, (tables,) budget] bf16 bit patterns: sorted N(0, 0.02^2) draws, 1 % of the tables with their end x20."""
    shape = (G, N, tables, 16) if tables else (G, N, 16)
    c = torch.randn(shape, generator=gen, device="cuda").mul_(0.02).sort(dim=-1).values
    if budget == 4:   # four interior columns: an outlier among four centroids would carry a quarter of a row
        return c[..., [1, 5, 10, 14]].contiguous().bfloat16().view(torch.int16)
    far = torch.rand(shape[:-1], generator=gen, device="cuda") < 0.01
    left = c[..., 0].abs() >= c[..., 15].abs()
    c[..., 0] = torch.where(far & left, c[..., 0] * 20, c[..., 0])
    c[..., 15] = torch.where(far & ~left, c[..., 15] * 20, c[..., 15])
    return c.bfloat16().view(torch.int16)


def _rotation(gen, H):
    """A dense random orthogonal matrix: sign flips and normalised Sylvester matrices in turn, formed in float64."""
    R = torch.eye(H, dtype=torch.float64, device="cuda")
    for _ in range(3):
        sign = torch.randint(0, 2, (H, 1), generator=gen, device="cuda").double().mul_(2).sub_(1)
        R.mul_(sign)
        n = 1
        while n < H:   # R <- H_n-butterfly of R, along the rows
            v = R.view(H // (2 * n), 2, n, H)
            a = v[:, 0] + v[:, 1]
            torch.sub(v[:, 0], v[:, 1], out=v[:, 1])
            v[:, 0] = a
            n *= 2
        R.div_(math.sqrt(H))
    return R.float()


def _zipf_bias(c):
    """Router biases by popularity rank: tau log p, tau as in synth.zipf_bias."""
    tau = math.sqrt((c.H - c.n_outliers + c.n_outliers * c.outlier_scale ** 2) / c.H) * math.sqrt(6.0) / math.pi
    p = [(r + 1.0) ** -c.zipf_s for r in range(c.E)]
    return [tau * math.log(v / sum(p)) for v in p]


def _inputs(case, seed):
    c = _config(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * int(seed) + 17)
    X = torch.randn((c.T, c.H), generator=gen, device="cuda")
    X[:, torch.randperm(c.H, generator=gen, device="cuda")[:c.n_outliers]] *= c.outlier_scale
    R = None if c.r_hadamard else _rotation(gen, c.H)
    Wr = torch.randn((c.E, c.H), generator=gen, device="cuda") / math.sqrt(c.H)
    bias = None
    if c.zipf_s > 0:   # the experts' popularity follows Zipf's law
        bias = torch.tensor(_zipf_bias(c), device="cuda")[torch.randperm(c.E, generator=gen, device="cuda")]
    G, per_byte = c.n_groups, 8 // c.index_bits
    budget = 1 << c.index_bits
    weights = []
    for N, K in ((2 * c.I, c.H), (c.H, c.I)):   # gate/up (rows interleaved), down
        idx = torch.randint(0, 256, (G, N, K // per_byte), dtype=torch.uint8, generator=gen, device="cuda")
        weights.append((idx, _centroids(gen, G, N, -(-K // c.group_k) if c.group_k else 0, budget)))
    return c, X, R, Wr, bias, weights


def prepare(case, seed):
    c, X, R, Wr, bias, weights = _inputs(case, seed)
    gate_up, down = (binding.DeviceCodebook(i, t, keep_canonical=False, group_k=c.group_k, index_bits=c.index_bits)
                     for i, t in weights)
    return {"layer": binding.DeviceLayer(c, R, Wr, bias, gate_up, down), "X": X}


def run(state):
    return binding.cq_moe_forward(state["layer"], state["X"])


# ------------------------------------------------------------------------------------------------
# what a call cannot do without
# ------------------------------------------------------------------------------------------------
def _active(c):
    """Routed experts that at least one token selects, for one draw of the router's distribution: the few outlier
    channels carry most of a token's norm, so the logits of all tokens lie close to a space of that many dimensions."""
    gen = torch.Generator().manual_seed(c.T)
    far = torch.randn((c.T, c.n_outliers), generator=gen) * c.outlier_scale
    logits = far @ torch.randn((c.n_outliers, c.E), generator=gen) / math.sqrt(c.H)
    logits += torch.randn((c.T, c.E), generator=gen) * math.sqrt(1.0 - c.n_outliers / c.H)
    if c.zipf_s > 0:
        logits += torch.tensor(_zipf_bias(c))
    return torch.topk(logits, c.top_k, dim=1).indices.unique().numel()


def work(case):
    c = _config(case)
    groups = _active(c) + c.S
    tables = [-(-K // c.group_k) if c.group_k else 1 for K in (c.H, c.I)]
    weights = sum(N * (K * c.index_bits // 8 + t * (2 << c.index_bits))
                  for N, K, t in ((2 * c.I, c.H, tables[0]), (c.H, c.I, tables[1])))
    rows = c.T * (c.top_k + c.S)
    rotation = 0 if c.r_hadamard else 1
    flops = 2.0 * rotation * c.T * c.H * c.H + 2.0 * c.T * c.H * c.E + 6.0 * rows * c.H * c.I
    nbytes = groups * weights + rotation * 4.0 * c.H * c.H + 4.0 * c.E * c.H + 8.0 * c.T * c.H
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Measured on the path itself, against float64 and with the rotation summed in another order: 8-bit codes 3e-4
    (f16 rounding of the intermediate), 4-bit codes 1.2e-3 (codes at a rounding tie, each of which moves its token's
    outputs by one step: up to 0.6 of the result's root mean square in a token of large scale)."""
    return {"rel": 1.2e-3, "max": 0.2} if case["act_bits"] == 8 else {"rel": 4.8e-3, "max": 0.95}


# ------------------------------------------------------------------------------------------------
# the layer in float64
# ------------------------------------------------------------------------------------------------
def _hadamard(n):
    """The matrix of the online-Hadamard variant (include/cq.h): Sylvester's, or Paley's of order 12, 28 or 44 times it."""
    odd = n
    while odd % 2 == 0:
        odd //= 2
    m = 1 if odd == 1 else 4 * odd
    p = n // m
    S = torch.ones(1, 1, dtype=torch.float64)
    while S.shape[0] < p:
        S = torch.cat([torch.cat([S, S], 1), torch.cat([S, -S], 1)], 0)
    if m == 1:
        return torch.ones(1, 1, dtype=torch.float64), S
    q = 13 if m == 28 else m - 1
    squares = {(a * a) % q for a in range(1, q)}
    chi = lambda v: 0.0 if v % q == 0 else 1.0 if v % q in squares else -1.0  # noqa: E731
    C = torch.zeros(q + 1, q + 1, dtype=torch.float64)
    C[0, 1:] = 1.0
    for i in range(q):
        C[i + 1, 0] = 1.0 if m == 28 else -1.0
        for j in range(q):
            C[i + 1, j + 1] = chi(i - j) if m == 28 else chi(j - i)
    one = torch.eye(q + 1, dtype=torch.float64)
    if m == 28:
        return torch.kron(C, torch.tensor([[1.0, 1.0], [1.0, -1.0]], dtype=torch.float64)) + \
            torch.kron(one, torch.tensor([[1.0, -1.0], [-1.0, -1.0]], dtype=torch.float64)), S
    return one + C, S


def _transform(x):
    """Rows times H_n / sqrt(n)."""
    n = x.shape[1]
    Hm, S = (v.to(x.device) for v in _hadamard(n))
    m, p = Hm.shape[0], S.shape[0]
    y = (x.reshape(-1, p) @ S).view(-1, m, p)
    y = (y.transpose(1, 2).reshape(-1, m) @ Hm).view(-1, p, m).transpose(1, 2)
    return y.reshape(-1, n) / math.sqrt(n)


def _quantized(x, bits):
    """Rows after the symmetric integer quantizer: codes times scale."""
    qmax = 2 ** (bits - 1) - 1
    s = x.abs().amax(dim=1, keepdim=True) / qmax
    s = torch.where(s == 0, torch.ones_like(s), s)
    return torch.clamp(torch.round(x / s), -qmax, qmax) * s


def _dense(idx, cent, c):
    """One group's matrix [N, K] in float64."""
    N = idx.shape[0]
    b = idx.int()
    parts = [(b >> s) & ((1 << c.index_bits) - 1) for s in range(0, 8, c.index_bits)]
    k = torch.stack(parts, dim=-1).view(N, -1).long()
    t = cent.view(torch.bfloat16).double()
    if not c.group_k:
        return torch.gather(t, 1, k)
    return torch.cat([torch.gather(t[:, j], 1, k[:, j * c.group_k:(j + 1) * c.group_k]) for j in range(t.shape[1])], 1)


def exact(case, seed):
    c, X, R, Wr, bias, ((gi, gc), (di, dc)) = _inputs(case, seed)
    XR = _transform(X.double()) if c.r_hadamard else X.double() @ R.double()
    a = _quantized(XR, c.act_bits)
    logits = XR @ Wr.double().T
    if bias is not None:
        logits = logits + bias.double()
    top, ids = torch.sort(logits, dim=1, descending=True, stable=True)
    w = torch.softmax(top[:, :c.top_k], dim=1)
    ids = ids[:, :c.top_k]
    Y = torch.zeros((c.T, c.H), dtype=torch.float64, device="cuda")
    for g in range(c.n_groups):
        if g < c.E:
            tok, slot = (ids == g).nonzero(as_tuple=True)
            if tok.numel() == 0:
                continue
            weight = w[tok, slot].unsqueeze(1)
        else:
            tok, weight = torch.arange(c.T, device="cuda"), 1.0
        gu = a[tok] @ _dense(gi[g], gc[g], c).T
        h = gu[:, 0::2] * torch.sigmoid(gu[:, 0::2]) * gu[:, 1::2]
        if c.h_bits:
            h = _quantized(_transform(h), c.h_bits)
        Y.index_add_(0, tok, weight * (h @ _dense(di[g], dc[g], c).T))
    return Y
