"""The measured workloads of the LookupFFN forward pass.

A case is one call of a public entry point on a batch that is already in device memory: the hash constants and the
learned tables are prepared once, as a serving program does when it loads a model, and the scratch and output
buffers are kept from call to call.  Field by field:

  entry    "plain" | "weighted" | "probes": lookupffn_forward[_weighted, _probes]; "bh" | "bh_weighted":
           lookupffn_forward_bh[_weighted]; "stack": lookupffn_forward_stack (chained layers, one launch)
  n, d     tokens of the batch, input width (padded to d_pad, the next power of two)
  k, tau   tables, code bits (2^tau rows a table);  d_out: row width
  rounds   sign-diagonal rounds, or factors of the block-diagonal hash;  block: its block size (0: sign diagonals)
  layers   chained layers (1 except for "stack")
  x, table, y   storage types "f32" | "bf16" | "f16";  prepared: tables in the layout lookupffn_prepare_tables writes
"""
from __future__ import annotations

import math

import torch

from paper_2403_07221_amd import binding as B

_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_BYTES = {"f32": 4, "bf16": 2, "f16": 2}
_ENTRY = {"plain": B.lookupffn_forward, "weighted": B.lookupffn_forward_weighted, "probes": B.lookupffn_forward_probes,
          "bh": B.lookupffn_forward_bh, "bh_weighted": B.lookupffn_forward_bh_weighted}


def _case(name, entry, n, d, k, tau, d_out, rounds, block=0, layers=1, x="f32", table="f32", y="f32", prepared=True):
    case = {"entry": entry, "n": n, "d": d, "k": k, "tau": tau, "d_out": d_out, "rounds": rounds, "block": block,
            "layers": layers, "x": x, "table": table, "y": y, "prepared": prepared}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # one call of a very small layer: launches and the host path decide
        _case("tiny_layer", "plain", 64, 64, 8, 8, 64, 2),
        # decoding eight sequences at once through twelve chained base-size layers: latency
        _case("decode_chain_12_layers", "stack", 8, 768, 96, 8, 768, 3, layers=12),
        # a small serving batch in the form the paper's experiments use (block-diagonal hash, weighted gather)
        _case("serve_128_bh_weighted", "bh_weighted", 128, 768, 96, 8, 768, 4, block=64),
        # a ragged prompt with odd sizes, half tables as they came from a checkpoint, outputs kept in half
        _case("ragged_f16_weighted", "weighted", 1001, 700, 97, 7, 648, 3, x="f16", table="f16", y="f16",
              prepared=False),
        # the headline layer: base-size encoder, 16384 tokens
        _case("base_layer", "plain", 16384, 768, 96, 8, 768, 3),
        # the same layer with the weighted gather
        _case("base_layer_weighted", "weighted", 16384, 768, 96, 8, 768, 3),
        # the same layer with the soft-max neighbourhood of each row (nine rows a table)
        _case("base_layer_probes", "probes", 16384, 768, 96, 8, 768, 3),
        # the same layer hashed with the cheapest block-diagonal factors
        _case("base_layer_bh16", "bh", 16384, 768, 96, 8, 768, 4, block=16),
        # bulk encoding, everything stored in bf16
        _case("bulk_bf16", "plain", 65536, 768, 96, 8, 768, 3, x="bf16", table="bf16", y="bf16"),
        # large-size layer: 512 MiB of tables of 1024 rows
        _case("large_layer_tau10", "plain", 16384, 1024, 128, 10, 1024, 3),
        # the paper's small model (many tables), at the batch of its latency study
        _case("small_model_h256", "plain", 32768, 512, 256, 8, 512, 3),
        # the paper's base-size experiment: block-diagonal hash, 512-row tables, weighted gather
        _case("base_tau9_bh64_weighted", "bh_weighted", 32768, 768, 170, 9, 768, 4, block=64),
    ]


def _d_pad(d):
    p = 1
    while p < d:
        p <<= 1
    return p


def _projections(case):
    return -(-case["k"] * case["tau"] // _d_pad(case["d"]))


def _rows_per_lookup(case):
    return 1 + case["tau"] if case["entry"] == "probes" else 1


def _rough_us(case):
    """A rough time of one pass (microseconds), to keep drawn cases below the largest listed one."""
    n, layers = case["n"], case["layers"]
    gathered = n * case["k"] * _rows_per_lookup(case) * case["d_out"] * 4 * layers
    staged = case["prepared"] and 7 <= case["tau"] <= 10
    tables = case["k"] * 2 ** case["tau"] * case["d_out"] * 4 * layers
    if case["block"]:
        hash_us = n * _projections(case) * case["rounds"] * _d_pad(case["d"]) * (2 * case["block"] + 64) / 50e6
    else:
        hash_us = n * _projections(case) * case["rounds"] * _d_pad(case["d"]) * 10 / 15e6
    return 10 + gathered / (30e6 if staged else 12e6) + tables / 3e6 + hash_us


def draw(rng):
    """One more case of the same ranges: 1 to 65536 tokens, rows of 32 to 1024, 4 to 256 tables of 2^4 to 2^11 rows."""
    while True:
        entry = rng.choice(["plain", "plain", "plain", "weighted", "weighted", "probes", "bh", "bh_weighted", "stack"])
        stack, bh = entry == "stack", entry.startswith("bh")
        n = int(round(2 ** rng.uniform(0, 5 if stack else 16)))
        if stack:
            d = rng.choice([520, 640, 768, 896, 1024])
        elif bh:
            d = rng.choice([64, 256, 512, 768, 1024, rng.randrange(65, 1025)])
        else:
            d = rng.choice([64, 256, 512, 768, 768, 1024, rng.randrange(48, 1025)])
        d_out = d if stack else rng.choice([64, 512, 768, 1024, 8 * rng.randrange(4, 129)])
        k = rng.choice([8, 96, 128, 170, int(round(2 ** rng.uniform(2, 8)))])
        tau = rng.choice([7, 8, 8, 8, 9, 10, rng.randrange(4, 12)])
        block = rng.choice([16, 32, 64]) if bh else 0
        table = rng.choice(["f32", "f32", "bf16", "f16"])
        case = _case(None, entry, n, d, k, tau, d_out, 4 if bh else rng.choice([2, 3, 3, 3, 4]), block=block,
                     layers=rng.choice([2, 6, 12]) if stack else 1, x=rng.choice(["f32", "f32", "bf16", "f16"]),
                     table=table, y=rng.choice(["f32", "f32", "f32", "bf16", "f16"]),
                     prepared=rng.random() < 0.85)
        if k * 2 ** tau * d_out * 4 <= 600e6 and _rough_us(case) <= 900:
            return case


def prepare(case, seed):
    """Activations N(0, 1), tables N(0, 0.02^2), Rademacher sign diagonals, factor entries N(0, 1/block): with a
    random rotation the codes are uniform over the rows, as an untrained or well-balanced hash makes them."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    n, d, k, tau, d_out = case["n"], case["d"], case["k"], case["tau"], case["d_out"]
    d_pad, P = _d_pad(d), _projections(case)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)

    B.lookupffn_init()
    hashes, tables = [], []
    for _ in range(case["layers"]):
        if case["block"]:
            b = case["block"]
            factors = normal(P, case["rounds"], d_pad // b, b, b).mul_(1.0 / math.sqrt(b))
            hashes.append(B.lookupffn_prepare_bh(factors, d, k, tau))
        else:
            bits = torch.randint(0, 2, (P, case["rounds"], d_pad), generator=gen, device="cuda", dtype=torch.int8)
            hashes.append(bits.mul_(2).sub_(1))
        t = normal(k, 2 ** tau, d_out).mul_(0.02).to(_DTYPE[case["table"]])
        tables.append(B.lookupffn_prepare_tables(t) if case["prepared"] else t)
    state = {"entry": case["entry"], "x": normal(n, d).to(_DTYPE[case["x"]]), "hashes": hashes, "tables": tables,
             "y": torch.empty((n, d_out), dtype=_DTYPE[case["y"]], device="cuda")}
    if case["entry"] == "weighted":
        size = B.lookupffn_workspace_bytes_weighted(n, k)
    elif case["entry"] == "probes":
        size = B.lookupffn_workspace_bytes_probes(n, k, tau)
    elif case["entry"] == "bh":
        size = B.lookupffn_workspace_bytes_bh(n, d, k, tau, B.PREPARED | case["block"], case["rounds"])
    elif case["entry"] == "bh_weighted":
        size = B.lookupffn_workspace_bytes_bh_weighted(n, d, k, tau, B.PREPARED | case["block"], case["rounds"])
    else:
        size = B.lookupffn_workspace_bytes(n, k)
    state["workspace"] = torch.empty(max(size, 256), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    if state["entry"] == "stack":
        return B.lookupffn_forward_stack(state["x"], state["hashes"], state["tables"], y=state["y"])
    return _ENTRY[state["entry"]](state["x"], state["hashes"][0], state["tables"][0], y=state["y"],
                                  workspace=state["workspace"])


def work(case):
    """Compulsory bytes (x, the rows touched at most once, the hash constants, y) and arithmetic of one pass."""
    n, d, k, d_out, layers = case["n"], case["d"], case["k"], case["d_out"], case["layers"]
    d_pad, P, rpl = _d_pad(d), _projections(case), _rows_per_lookup(case)
    row_bytes = d_out * (4 if case["prepared"] else _BYTES[case["table"]])
    rows = min(k * 2 ** case["tau"], n * k * rpl)
    const = P * case["rounds"] * d_pad * (4 * case["block"] if case["block"] else 1)
    nbytes = n * d * _BYTES[case["x"]] + n * d_out * _BYTES[case["y"]] + layers * (rows * row_bytes + const)
    transform = P * case["rounds"] * d_pad * (math.log2(d_pad) + 2 * case["block"])
    gather = k * rpl * d_out * (1 if case["entry"] in ("plain", "bh", "stack") else 2)
    return {"bytes": int(nbytes), "flops": int(n * layers * (transform + gather))}


def tolerance(case):
    # The codes are defined bit for bit (order of the butterflies and of the products), so they do not differ between
    # correct implementations; what may differ is the order and fusing of the fp32 sums and the weights' exp2 and
    # reciprocal, and one rounding to y's type.  Measured against the same pass with its sums in 64 bits, largest of
    # the listed and 24 drawn cases: fp32 y 6.8e-7 of the 2-norm and 4.4e-6 for one element; bf16 y 1.7e-3 and 3.9e-3,
    # half y 2.1e-4 and 4.9e-4 (the rounding of the stored value).
    if case["y"] == "f32":
        return {"rel": 2.5e-6, "max": 2e-5}
    if case["y"] == "bf16":
        return {"rel": 4e-3, "max": 1.6e-2}
    return {"rel": 5e-4, "max": 2e-3}
