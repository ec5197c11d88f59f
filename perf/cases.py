"""Cases of the optimizer step, the save window and the checkpoint load.

What a training program has this library do: one fused optimizer step per
training step (the bulk of its calls), now and then a save window of K steps
with its drain and restore, and after a crash one load.  Sizes are the
repository's own workloads and one rank's share of them, the sizes of its
smoke check and tests, and generic odd ones between.  State arrays are
ordinary torch allocations, as Session makes them.
"""
import math
import os
import tempfile

import numpy as np
import torch

from paper_2511_07035_amd import Session, gockpt_arena_layout_ex, gockpt_plan_bounds, gockpt_write_checkpoint

LR = 1e-4
BETA1, BETA2, EPS, DECAY = 0.9, 0.999, 1e-8, 0.01  # the Session defaults
T0 = 1000  # steps taken before the measured ones
SCALE0 = 65536.0  # loss scale of the dynamic cases


def listed():
    return [
        # the smallest calls: a small model or a late, ragged shard; launches count
        {"name": "step_64k", "kind": "step", "n": 65560, "grad": "bf16"},
        # the same captured once in a graph and replayed, as launch-bound loops do
        {"name": "step_256k_graph", "kind": "step", "n": 262147, "grad": "bf16", "graph": True},
        # fp16 training with dynamic loss scaling, a small odd size
        {"name": "step_1m_fp16", "kind": "step", "n": 1048579, "grad": "fp16", "dynamic": True},
        # the flat 16.7M workload
        {"name": "step_16m", "kind": "step", "n": 16777216, "grad": "bf16"},
        # gradients scanned bucket by bucket beside the backward
        {"name": "step_124m_buckets", "kind": "step", "n": 124439808, "grad": "bf16", "buckets": 8},
        # the caller's scaler has tested the gradients, no norm: no read of them before the update
        {"name": "step_350m_flag", "kind": "step", "n": 350000003, "grad": "fp16", "dynamic": True, "flag": True},
        # one rank of eight of the 13B layout: the largest state a rank holds
        {"name": "step_13b_rank", "kind": "step", "n": 1626982912, "grad": "bf16"},
        # the smallest window: the smoke check's size
        {"name": "window_64k", "kind": "window", "n": 65560, "grad": "bf16", "K": 4, "ring_mib": 1, "plan": 2},
        # the flat 16.7M workload's window
        {"name": "window_16m", "kind": "window", "n": 16777216, "grad": "bf16", "K": 4, "ring_mib": 256, "plan": 2},
        # fp16 with a skipped step, a ring smaller than a step's pack list, restore into the caller's arrays
        {"name": "window_30m_fp16", "kind": "window", "n": 30000003, "grad": "fp16", "dynamic": True, "K": 8,
         "ring_mib": 32, "plan": 0, "inf_step": 3, "out": True},
        # an arena larger than the host pins: staging slots and replay inside the window
        {"name": "window_16m_staged", "kind": "window", "n": 16777219, "grad": "bf16", "K": 8, "ring_mib": 64,
         "plan": 2, "pageable": True, "replay_every": 2},
        # resume after a crash: the files in the page cache
        {"name": "load_8m", "kind": "load", "n": 8388611, "grad": "bf16"},
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choices(["step", "window", "load"], [6, 3, 1])[0]
    grad = rng.choice(["bf16", "fp16"])
    c = {"kind": kind, "grad": grad, "dynamic": grad == "fp16"}
    if kind == "step":
        c["n"] = _log_uniform(rng, 16384, 1.6e9)
        option = rng.choice(["plain", "plain", "graph", "flag", "buckets"])
        if option == "buckets":
            c["buckets"] = rng.randint(2, 8)
        elif option != "plain":
            c[option] = True
    elif kind == "window":
        c["n"] = _log_uniform(rng, 16384, 2.4e7)
        c["K"] = rng.randint(1, 8)
        c["ring_mib"] = rng.choice([1, 16, 256])
        c["plan"] = rng.randint(0, 2)
        c["out"] = rng.random() < 0.5
        if c["K"] >= 4 and rng.random() < 0.3:
            c["pageable"], c["replay_every"] = True, 2
    else:
        c["n"] = _log_uniform(rng, 16384, 8.3e6)
    return c


def _dtype(case):
    return torch.float16 if case["grad"] == "fp16" else torch.bfloat16


def _inputs(case, seed):
    """State (master, exp_avg, exp_avg_sq) and the 16-bit gradients of each step."""
    n, dev = case["n"], "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 7919 + 17)
    p = torch.empty(n, device=dev).normal_(0.0, 0.02, generator=gen)
    m = torch.empty(n, device=dev).normal_(0.0, 2e-4, generator=gen)
    v = torch.empty(n, device=dev).normal_(0.0, 1e-3, generator=gen).square_()
    grads = []
    for s in range(1, (case["K"] if case["kind"] == "window" else 1) + 1):
        g = torch.empty(n, dtype=_dtype(case), device=dev)
        for a in range(0, n, 1 << 28):
            part = g[a:a + (1 << 28)]
            sigma = 1e-3 * (SCALE0 if case.get("dynamic") else 1.0)
            part.copy_(torch.empty(part.numel(), device=dev).normal_(0.0, sigma, generator=gen))
        if case.get("inf_step") == s:
            g[n // 3] = float("inf")
        grads.append(g)
    return p, m, v, grads


class _State:
    """What the program holds; the session closes with it."""

    sess = graph = tmp = None

    def __del__(self):
        self.graph = None
        if self.sess is not None:
            self.sess.close()


class _Held:
    """A view of the session's host arena that keeps the session open."""

    def __init__(self, view, owner):
        self.__array_interface__ = view.__array_interface__
        self.owner = owner


def prepare(case, seed):
    n, K = case["n"], case.get("K", 0)
    st = _State()
    st.case = case
    p, m, v, grads = _inputs(case, seed)
    dyn = bool(case.get("dynamic"))
    kw = dict(dynamic_scale=dyn, init_scale=SCALE0 if dyn else 1.0, growth_interval=2000, init_step=T0,
              grad_dtype=case["grad"], ring_bytes=case.get("ring_mib", 0) << 20)
    if case["kind"] == "load":
        st.sess = Session(n, **kw)
        st.tmp = tempfile.TemporaryDirectory(prefix="gockpt_case_")
        st.path = os.path.join(st.tmp.name, "step%d" % T0)
        gockpt_write_checkpoint(st.path, p.cpu().numpy(), m.cpu().numpy(), v.cpu().numpy(), t=T0,
                                scale=SCALE0 if dyn else 1.0)
        st.sess.ensure_arena(12 * n)
        torch.cuda.synchronize()
        return st
    if case.get("flag"):
        kw.update(found_inf=torch.zeros(1, device="cuda"), grad_norm=False)
    if K:
        kw.update(copy_bytes=4 << 20, staging_bytes=(64 << 20) if case.get("pageable") else 0)
    st.sess = Session(n, master=p, exp_avg=m, exp_avg_sq=v, weight=p.to(torch.bfloat16),
                      grad=grads[0].clone() if K else grads[0], **kw)
    if K:
        st.bank = grads
        st.bounds = gockpt_plan_bounds(K, n)
        lay, _ = gockpt_arena_layout_ex(K, st.bounds, n, case.get("replay_every", 0))
        st.sess.ensure_arena(lay.total, bool(case.get("pageable")))
        st.out = None
        if case.get("out"):
            st.out = tuple(np.zeros(n, t) for t in (np.float32, np.float32, np.float32, np.uint16))
    if case.get("buckets"):
        st.side = torch.cuda.Stream()
        ends = [n * k // case["buckets"] // 8 * 8 for k in range(case["buckets"])] + [n]
        st.buckets = list(zip(ends[:-1], ends[1:]))[::-1]  # the backward finishes the last layers first
    torch.cuda.synchronize()
    if case.get("graph"):
        st.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st.graph, stream=st.sess.compute):
            st.sess.step(LR)
        torch.cuda.synchronize()
    return st


def run(st):
    case, sess = st.case, st.sess
    if case["kind"] == "load":
        info = sess.load(st.path)
        return {"state": (sess.master, sess.exp_avg, sess.exp_avg_sq), "weight": sess.weight, "t": int(info.t)}
    if case["kind"] == "step":
        if st.graph is not None:
            with torch.cuda.stream(sess.compute):
                st.graph.replay()
        else:
            sess.backward_begin()
            if case.get("buckets"):
                for k, (a, b) in enumerate(st.buckets):
                    if k + 1 < len(st.buckets):
                        st.side.wait_stream(sess.compute)  # the bucket's gradients are written there
                        sess.scan_grads(a, b, stream=st.side)
                    else:
                        sess.scan_grads(a, b)
            sess.step(LR)
        return {"state": (sess.master, sess.exp_avg, sess.exp_avg_sq), "weight": sess.weight}
    sess.begin_window(st.bounds, replay_every=case.get("replay_every", 0), pageable=bool(case.get("pageable")),
                      late_plan=case["plan"])
    for g in st.bank:
        sess.backward_begin()
        with torch.cuda.stream(sess.compute):
            sess.grad.copy_(g)  # the backward writes the gradients
        sess.step(LR)
    sess.drain()
    rec = sess.records()
    meta = sess.restore(out=st.out)
    host = st.out[:3] if st.out else tuple(np.asarray(_Held(a, st)) for a in sess.arena_state())
    return {"state": (sess.master, sess.exp_avg, sess.exp_avg_sq), "weight": sess.weight, "host": host,
            "host_weight": st.out[3] if st.out else 0, "gnorm2": rec["gnorm2"].copy(), "skip": rec["skip"].copy(),
            "t": int(meta.t)}


def exact(case, seed):
    """AdamW in float64 from the same inputs."""
    p, m, v, grads = (x if isinstance(x, list) else x.double() for x in _inputs(case, seed))
    gnorm2, t, scale = [], T0, SCALE0 if case.get("dynamic") else 1.0
    lr = float(np.float32(LR))
    for g in grads if case["kind"] != "load" else []:
        norm = 0.0
        finite = bool(torch.isfinite(g).all())
        t += finite
        bc1, bc2 = 1.0 - BETA1 ** t, 1.0 - BETA2 ** t
        for a in range(0, case["n"], 1 << 27):
            q = slice(a, a + (1 << 27))
            x = g[q].double() / scale
            norm += float(x.square().sum())
            if not finite:
                continue
            m[q].mul_(BETA1).add_(x, alpha=1.0 - BETA1)
            v[q].mul_(BETA2).addcmul_(x, x, value=1.0 - BETA2)
            step = m[q] / (v[q].sqrt() / math.sqrt(bc2) + EPS)
            p[q].mul_(1.0 - lr * DECAY).sub_(step, alpha=lr / bc1)
        gnorm2.append(norm)
        if not finite:
            scale *= 0.5
    out = {"state": (p, m, v), "weight": p}
    if case["kind"] == "load":
        out["t"] = None
    elif case["kind"] == "window":
        out.update(host=(p, m, v), host_weight=None, gnorm2=np.array(gnorm2), skip=None, t=None)
    return out


def work(case):
    n = case["n"]
    if case["kind"] == "load":  # the file's 12 bytes an element to the device, and its bf16 weights
        return {"bytes": 26 * n, "flops": 0}
    step = 28 * n  # gradient, master and moments in; master, moments and weight out
    if case["kind"] == "step":
        return {"bytes": step, "flops": 18 * n}
    K = case["K"]
    b = [int(x) for x in gockpt_plan_bounds(K, n)]
    sent = 12 * n + 2 * sum(b[:K])  # the parts, and the gradients of parts already sent, to the host
    return {"bytes": K * (step + 4 * n) + sent + 12 * n, "flops": 18 * n * K}


def tolerance(case):
    # a step is one stated fp32 operation after the other: the same bits.  In
    # a window only the gradient norm, a sum, may differ: measured 1.5e-8
    # against float64.
    if case["kind"] == "window":
        return {"rel": 6e-8, "max": 6e-7}
    return "exact"
