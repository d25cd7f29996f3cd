"""The work a user of this library has it do, as cases that can be timed: requests served by one model on its share of
the compute units, mixes of co-located models served in closed loop, and the allocation solve that precedes serving.

A case is a dict of plain values.  Serving cases:
  models    networks separated by "+", one worker each (see _NETS)
  batch     samples per request
  size      image side of the CNNs / sequence length of the encoders, separated by "+" like the models
  dtype     storage type of each model
  cus       compute units of each worker's stream
  cus2      0, or the compute units of a second stream that every other kernel group runs on (a table that switches)
  requests  requests per worker in one pass: 1 = submitted and waited for, more = closed loop with two in flight
  tuned     whether the launch plans are chosen by measurement after loading (eclip_model_tune)
Allocation cases (`kind` = "allocate"): units of each worker, CU configurations, switch budget and limits of the model.

Weights are synthetic (He-normal CNNs, N(0, 0.02) encoders) and fixed per network, as a server loads a model once;
request inputs come from the seed.
"""
from __future__ import annotations

import contextlib
import json
import math
import weakref
from concurrent.futures import ThreadPoolExecutor
from unittest import mock

import numpy as np
import torch

import paper_2506_12598_amd as ec
import workloads as wl
import workloads.graphs as graphs

_DT = {"f32": wl.DT_F32, "bf16": wl.DT_BF16, "f16": wl.DT_F16}
_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}

_NETS = {
    "tiny_cnn": lambda s, d: graphs.tiny_cnn(dtype=d, hw=s),
    "resnet18": lambda s, d: graphs.resnet(18, dtype=d, hw=s),
    "resnet50": lambda s, d: graphs.resnet(50, dtype=d, hw=s),
    "resnet152": lambda s, d: graphs.resnet(152, dtype=d, hw=s, res_scale=0.25),
    "vgg16": lambda s, d: graphs.vgg16(dtype=d, hw=s),
    "mobilenetv2": lambda s, d: graphs.mobilenetv2(dtype=d, hw=s),
    "densenet": lambda s, d: graphs.densenet(dtype=d, hw=s),
    "resnext": lambda s, d: graphs.resnext(dtype=d, hw=s, res_scale=0.5),
    "shufflenet": lambda s, d: graphs.shufflenet(dtype=d, hw=s),
    "bert_base": lambda s, d: graphs.bert(seq=s, dtype=d),
    "bert_large": lambda s, d: graphs.bert(24, 1024, 16, 4096, s, dtype=d),
    "albert": lambda s, d: graphs.albert(seq=s, dtype=d),
}


def _serve(name, models, batch, size, dtype, cus, cus2=0, requests=1, tuned=False):
    return {"name": name, "kind": "serve", "models": models, "batch": batch, "size": size, "dtype": dtype, "cus": cus, "cus2": cus2,
            "requests": requests, "tuned": tuned}


def listed():
    return [
        # the smallest request there is: a four-layer float32 CNN, all launch and wait
        _serve("tiny_cnn_f32_b1", "tiny_cnn", "1", "32", "f32", "64"),
        # the classic co-location: two light classifiers at batch 1, each on half of the GPU
        _serve("resnet18_pair_b1", "resnet18+resnet18", "1+1", "224+224", "bf16+bf16", "128+128", requests=8),
        # one latency-critical classifier whose kernel groups alternate between two shares (the table of Sec. III-B)
        _serve("resnet50_b1_switching", "resnet50", "1", "224", "bf16", "256", cus2=128),
        # depthwise and pointwise layers, float16, an odd batch
        _serve("mobilenetv2_f16_b3", "mobilenetv2", "3", "224", "f16", "192"),
        # wide convolutions and 250 MB of classifier weights, a full batch
        _serve("vgg16_b8", "vgg16", "8", "224", "bf16", "256"),
        # one short sentence at batch 1
        _serve("bert_base_f16_b1", "bert_base", "1", "128", "f16", "256"),
        # a ragged sentence length and batch
        _serve("bert_base_bf16_b5_s201", "bert_base", "5", "201", "bf16", "160"),
        # a large encoder on the share it gets next to neighbours
        _serve("bert_large_b4_cu96", "bert_large", "4", "384", "bf16", "96"),
        # the second workload family at batch 1: shared-weight encoder + dense blocks ...
        _serve("albert_densenet_b1", "albert+densenet", "1+1", "128+224", "f16+bf16", "64+192", requests=4),
        # ... and grouped convolutions + channel shuffles, at a small image
        _serve("resnext_shufflenet_b2", "resnext+shufflenet", "2+2", "160+160", "bf16+bf16", "128+128", requests=4),
        # the stress mix the headline figure is quoted on, two requests per worker
        _serve("stress_mix", "bert_large+bert_large+bert_large+resnet152", "4+4+4+8", "384+384+384+224", "bf16+bf16+bf16+bf16",
               "96+96+96+112", requests=2, tuned=True),
        # choosing the shares of four workers from their latency tables, as a server does whenever its mix changes
        {"name": "allocate_4_workers", "kind": "allocate", "units": "8+8+8+4", "configs": 8, "switch_max": 14, "max_configs": 0,
         "switch_cost_ns": 0, "overlap": "excess"},
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_net(rng, net):
    """(batch, size, dtype) of a request to `net`."""
    if net == "tiny_cnn":
        return _spread(rng, 1, 8), _spread(rng, 16, 64), "f32"
    if net in ("bert_base", "albert"):
        return _spread(rng, 1, 8), _spread(rng, 17, 384), rng.choice(["f16", "bf16"])
    if net == "bert_large":
        return _spread(rng, 1, 4), _spread(rng, 64, 384), "bf16"
    return _spread(rng, 1, 8), rng.randint(64, 224), "f16" if net == "mobilenetv2" else "bf16"


def draw(rng):
    what = rng.random()
    if what < 0.08:
        n = rng.randint(2, 4)
        return {"kind": "allocate", "units": "+".join(str(rng.randint(3, 8)) for _ in range(n)), "configs": rng.randint(3, 8),
                "switch_max": rng.randint(2, 14), "max_configs": rng.choice([0, 0, 1, 2]), "switch_cost_ns": rng.choice([0, rng.randint(2000, 26000)]),
                "overlap": rng.choice(["excess", "literal", "table"])}
    if what < 0.3:
        # two or three light models next to each other on disjoint shares
        nets = [rng.choice(["resnet18", "resnet50", "mobilenetv2", "densenet", "resnext", "shufflenet", "bert_base", "albert"])
                for _ in range(rng.randint(2, 3))]
        sizes = [_draw_net(rng, n) for n in nets]
        cus = [16 * rng.randint(2, 16 // len(nets)) for _ in nets]
        c = _serve("", "+".join(nets), "+".join(str(s[0]) for s in sizes), "+".join(str(s[1]) for s in sizes), "+".join(s[2] for s in sizes),
                   "+".join(str(v) for v in cus), requests=rng.randint(2, 4))
    else:
        net = rng.choice(list(_NETS))
        b, size, dt = _draw_net(rng, net)
        cus = 16 * rng.randint(2, 16)
        c = _serve("", net, str(b), str(size), dt, str(cus), cus2=16 * rng.randint(2, 16) if rng.random() < 0.2 else 0)
    del c["name"]
    return c


# ---- networks ---------------------------------------------------------------------------------------------------
class _Shapes(graphs._Builder):
    """Builds a network's layer list and notes which weights it needs instead of drawing them one by one on the host."""

    made = None

    def __init__(self, *a):
        super().__init__(*a)
        self.specs = []
        _Shapes.made = self

    def _reserve(self, n, mean, std):
        off = self.n_elems
        self.specs.append((off, n, mean, std))
        self.n_elems += n + (-n) % 16
        return off

    def normal(self, shape, std):
        return self._reserve(int(np.prod(shape)), 0.0, float(std))

    def const(self, n, val):
        return self._reserve(n, float(val), 0.0)


_graphs_built = {}


def _network(net, size, dtype):
    """(Model without weight values, [(offset, elements, mean, std)], elements of the blob)"""
    key = (net, size, dtype)
    if key not in _graphs_built:
        with mock.patch.object(graphs, "_Builder", _Shapes):
            m = _NETS[net](size, _DT[dtype])
        _graphs_built[key] = (m, _Shapes.made.specs, _Shapes.made.n_elems)
    return _graphs_built[key]


def _weights(net, size, dtype):
    _, specs, n = _network(net, size, dtype)
    gen = torch.Generator("cuda").manual_seed(1234)
    blob = torch.zeros(max(16, n), dtype=_TORCH[dtype], device="cuda")
    for off, count, mean, std in specs:
        if std > 0:
            blob[off:off + count] = torch.randn(count, generator=gen, device="cuda").mul_(std).add_(mean).to(blob.dtype)
        else:
            blob[off:off + count] = mean
    return (blob.view(torch.int16) if dtype != "f32" else blob).cpu().numpy()


# ---- what a serving program keeps: one pool of streams, models loaded once ---------------------------------------
_loaded = {}                                   # loaded models wait on a pool without masked streams between servers
_parking = []


def _park():
    if not _parking:
        _parking.append(ec.Pool([(None, -1)]))
    return _parking[0]


class _Server:
    """The streams of one case and its models, one worker thread per model when there is more than one."""

    def __init__(self, case):
        nets, batch, size = case["models"].split("+"), case["batch"].split("+"), case["size"].split("+")
        dtype, cus = case["dtype"].split("+"), [int(v) for v in case["cus"].split("+")]
        total = _park().device_cus()
        masks = [(ec.eclip_mask_layout(total, 16, len(nets), w, c // 16), w) for w, c in enumerate(cus)]
        if case["cus2"]:
            masks.append((ec.eclip_mask_layout(total, 16, 1, 0, case["cus2"] // 16), 0))
        self.pool = ec.Pool(masks)
        self.workers, self.keys = [], []
        blobs = {}
        for w, (net, b, s, d) in enumerate(zip(nets, batch, size, dtype)):
            key = (net, int(b), int(s), d, bool(case["tuned"]), nets[:w].count(net))
            desc = _network(net, int(s), d)[0]
            h = _loaded.pop(key, None)
            if h is None:
                if (net, s, d) not in blobs:
                    blobs[net, s, d] = _weights(net, int(s), d)
                h = ec.Model(self.pool, desc, blobs[net, s, d], max_batch=int(b), max_inflight=2)
            else:
                h.rebind(self.pool)
            if case["tuned"]:
                h.tune(w, batch=int(b), iters=2)
            h.alloc_set([len(nets) if case["cus2"] and g % 2 else w for g in range(desc.n_groups)])
            self.workers.append((h, desc, int(b), d))
            self.keys.append(key)
        self.threads = ThreadPoolExecutor(len(nets)) if len(nets) > 1 else None

    def __del__(self):
        with contextlib.suppress(Exception):
            if self.threads:
                self.threads.shutdown()
            torch.cuda.synchronize()
            for key, (h, *_) in zip(self.keys, self.workers):
                h.rebind(_park())
                _loaded[key] = h
            self.pool.destroy()


_servers = weakref.WeakValueDictionary()       # one server per case while any of its states is in use


def _latency_tables(case, seed):
    """Latency of every unit at every configuration, ns: falls with the compute units down to a floor of its own."""
    r = np.random.default_rng(seed)
    configs = [16 * (16 * (i + 1) // case["configs"]) for i in range(case["configs"])]
    nk, beta = [], []
    for n in (int(v) for v in case["units"].split("+")):
        rows = []
        for _ in range(n):
            t, floor, noise = r.uniform(5e4, 6e5), r.uniform(0.1, 0.9), r.uniform(0.98, 1.02, len(configs))
            rows.append([int(t * max(floor, min(1.0, 64.0 / c)) * k) for c, k in zip(configs, noise)])
        nk.append([int(v) for v in r.integers(5, 26, n)])
        beta.append(rows)
    return configs, nk, beta


def prepare(case, seed):
    if case["kind"] == "allocate":
        configs, nk, beta = _latency_tables(case, seed)
        mode = {"excess": ec.OVERLAP_EXCESS, "literal": ec.OVERLAP_LITERAL, "table": ec.OVERLAP_TABLE}[case["overlap"]]
        more = {"alpha_ppm": [40_000 * i for i in range(32)], "granule": 32} if case["overlap"] == "table" else {}
        return {"allocate": (256, configs, nk, beta, case["switch_max"]),
                "options": dict(more, overlap_mode=mode, max_configs=case["max_configs"], switch_cost_ns=case["switch_cost_ns"])}
    key = json.dumps({k: v for k, v in case.items() if k != "name"}, sort_keys=True)
    server = _servers.get(key)
    if server is None:
        server = _servers[key] = _Server(case)
    gen = torch.Generator("cuda").manual_seed(int(seed))
    ins, outs = [], []
    for h, desc, b, d in server.workers:
        shape = (case["requests"],) + desc.in_shape(b)
        if desc.in_kind == wl.IN_TOKENS:
            x = torch.randint(0, desc.layers[0].aux0, shape, generator=gen, dtype=torch.int32, device="cuda")
        else:
            x = torch.randn(shape, generator=gen, device="cuda").to(_TORCH[d])
        ins.append(list(x))
        outs.append(list(torch.zeros((case["requests"],) + desc.out_shape(b), device="cuda")))
    return {"server": server, "in": ins, "out": outs}


def _closed_loop(model, batch, ins, outs):
    """One worker: its requests in order, two in flight."""
    flying = []
    for x, y in zip(ins, outs):
        if len(flying) == 2:
            flying.pop(0).wait()
        flying.append(model.submit(x.data_ptr(), y.data_ptr(), batch))
    for r in flying:
        r.wait()


def run(state):
    if "allocate" in state:
        table, objective, switches = ec.eclip_alloc_solve(*state["allocate"], **state["options"])
        return {"table": [np.array(t) for t in table], "switches": np.array(switches), "objective": [objective >> (32 * i) & 0xFFFFFFFF for i in range(4)]}
    server = state["server"]
    if server.threads is None:
        h, _, b, _ = server.workers[0]
        _closed_loop(h, b, state["in"][0], state["out"][0])
    else:
        jobs = [server.threads.submit(_closed_loop, h, b, x, y) for (h, _, b, _), x, y in zip(server.workers, state["in"], state["out"])]
        for j in jobs:
            j.result()
    return state["out"]


def work(case):
    """Weights once per pass and model, inputs and outputs once per request; of an embedding's tables the rows looked up."""
    if case["kind"] == "allocate":
        units = sum(int(v) for v in case["units"].split("+"))
        return {"bytes": 8.0 * units * case["configs"] + 8.0 * units, "flops": float(units * case["configs"])}
    nbytes = flops = 0.0
    for net, b, s, d in zip(*(case[k].split("+") for k in ("models", "batch", "size", "dtype"))):
        m, _, n = _network(net, int(s), d)
        b, e = int(b), 4 if d == "f32" else 2
        per_in = float(np.prod(m.in_shape(b))) * (4 if m.in_kind == wl.IN_TOKENS else e)
        if m.layers[0].op == wl.OP_EMBED:
            L = m.layers[0]
            n -= (L.aux0 + L.aux1 + 2) * L.c
            n += (b * L.w + L.w + 1) * L.c
        nbytes += float(n) * e + case["requests"] * (per_in + 4.0 * float(np.prod(m.out_shape(b))))
        flops += case["requests"] * b * m.flops_per_sample
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Activations are rounded to the storage type after every layer and the sums in between associate freely, so two correct
    implementations drift apart over the 20 to 170 layers of a network (24 normalised encoder layers in bf16: 1 %; CNNs and
    the shorter encoders: a few tenths); allocations are integers."""
    if case["kind"] == "allocate":
        return "exact"
    d = case["dtype"].split("+")
    return {"rel": (2e-2 if "bert_large" in case["models"] else 1e-2) if "bf16" in d else 5e-3 if "f16" in d else 1e-5}
