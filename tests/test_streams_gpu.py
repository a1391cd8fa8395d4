"""Two decodes on two streams at once.

The library keeps no state between calls (the allocation-free beam step's
per-GPU array aside, which is documented and not used here): cross-attention,
fused append + self-attention and the beam step of two different workloads,
issued step by step alternately on two streams so that their kernels overlap
on the GPU, give bit-identical outputs, tables and selections to the same
calls issued one workload after the other on one stream.
"""
import math
import sys

import numpy as np
import pytest
import torch

from cross_launch import bf16_kernel
from paper_2608_00938_amd import grace as G
from paper_2608_00938_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [
    W.custom("streams_a", B=4, M=300, H=30, d=64, steps=4, L=200, parents="uniform"),
    W.custom("streams_b", B=3, M=130, H=18, d=128, steps=3, L_lo=5, L_hi=260, parents="zipf",
             zipf_s=1.2),
]
V_TOK = 96   # beam-step vocabulary
K_SEL = 64   # beams selected per request


class _Decode:
    """All inputs and outputs of one workload's decode, allocated up front."""

    def __init__(self, wl, seed, dev):
        self.wl = wl
        inp = W.DecodeInputs(wl, seed, dev)
        self.ek, self.ev = inp.enc_kv
        self.off = inp.offsets_tensor()
        self.scale = 1.0 / math.sqrt(wl.d)
        T = wl.steps
        self.qc = [inp.step_tensor("q_cross", t) for t in range(T)]
        self.qs = [inp.step_tensor("q_self", t) for t in range(T)]
        self.kn = [inp.step_tensor("k_new", t) for t in range(T)]
        self.vn = [inp.step_tensor("v_new", t) for t in range(T)]
        self.par = [None if inp.parents(t) is None else torch.from_numpy(inp.parents(t)).to(dev)
                    for t in range(T)]
        R = wl.R
        self.logits = [W.beam_logits(seed, t, R, V_TOK, device=dev) for t in range(T)]
        self.prev = [torch.from_numpy(W.beam_prev_scores(seed, t, R)).to(dev) for t in range(T)]
        need = G.grace_beam_step_workspace_bytes(wl.B, wl.M, V_TOK)
        self.ws = torch.empty((max(need, 8),), dtype=torch.uint8, device=dev)
        self.reset(dev)

    def reset(self, dev):
        wl, T = self.wl, self.wl.steps
        shape = (wl.R, wl.H, wl.d)
        self.cache = G.KVCache(wl.B, wl.M, wl.H, wl.d, T, wl.torch_dtype, dev)
        self.xc = [torch.full(shape, float("nan"), dtype=wl.torch_dtype, device=dev) for _ in range(T)]
        self.xs = [torch.full(shape, float("nan"), dtype=wl.torch_dtype, device=dev) for _ in range(T)]
        self.tables = [torch.zeros((wl.R, T), dtype=torch.int32, device=dev) for _ in range(T)]
        self.sel = [tuple(torch.zeros((wl.B, K_SEL), dtype=dt, device=dev)
                          for dt in (torch.int32, torch.int32, torch.float32)) for _ in range(T)]

    def step(self, t):
        G.grace_cross_attn(self.qc[t], self.ek, self.ev, self.off, self.wl.M, self.scale,
                           out=self.xc[t])
        self.cache.append_attend(t, self.qs[t], self.kn[t], self.vn[t], self.par[t], self.scale,
                                 out=self.xs[t])
        self.tables[t].copy_(self.cache.table(t))
        p, tok, sc = self.sel[t]
        G.grace_beam_step(self.logits[t], self.prev[t], self.wl.B, self.wl.M, K_SEL,
                          parents=p, tokens=tok, scores=sc, workspace=self.ws)

    def results(self):
        out = {"xc": self.xc, "xs": self.xs, "tables": self.tables}
        out["sel"] = [t for s in self.sel for t in s]
        return {k: [x.clone() for x in v] for k, v in out.items()}


def test_two_streams_match_one_stream(gpu):
    for wl in CASES:   # the cross-attention kernel that keeps its keys in LDS for all waves
        assert bf16_kernel(wl.B, wl.M, wl.H, wl.d) == "whole"
    decs = [_Decode(wl, seed, gpu) for seed, wl in enumerate(CASES, start=41)]
    for d in decs:
        for t in range(d.wl.steps):
            d.step(t)
    torch.cuda.synchronize()
    serial = [d.results() for d in decs]
    for d in decs:
        assert int(d.cache.err_flag.item()) == 0
        d.reset(gpu)
    torch.cuda.synchronize()

    streams = [torch.cuda.Stream(device=gpu) for _ in decs]   # default priority
    for t in range(max(d.wl.steps for d in decs)):
        for d, s in zip(decs, streams):
            if t < d.wl.steps:
                with torch.cuda.stream(s):
                    d.step(t)
    for s in streams:
        s.synchronize()
    torch.cuda.synchronize()
    for d, ref in zip(decs, serial):
        got = d.results()
        print(f"{d.wl.name}: comparing {sum(len(v) for v in got.values())} tensors", flush=True)
        sys.stdout.flush()
        for key in ref:
            for i, (a, b) in enumerate(zip(ref[key], got[key])):
                assert not torch.isnan(b.float()).any() if b.is_floating_point() else True, (key, i)
                assert torch.equal(a, b), (d.wl.name, key, i)
