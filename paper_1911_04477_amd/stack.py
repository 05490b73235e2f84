"""The binarized VGG-small stack as a sequence of C-ABI calls (orchestration only).

Block order (every step runs in a HIP kernel of libbnn):
  conv -> int32 accumulators -> (2x2 max-pool on int32 when the block pools)
       -> fma(scale, acc, bias) -> fp32 map whose sign the next binarized layer takes.
Un-pooled blocks get the affine map from the GEMM store itself; pooled blocks from
the pool kernel.  The binarized FC flattens in NCHW order.
"""
from __future__ import annotations

from typing import Dict, List, Sequence

import numpy as np
import torch

from . import binding as B


class VggStack:
    def __init__(self, layers: Sequence, params: Sequence[Dict[str, np.ndarray]], batch: int, device="cuda:0"):
        self.layers = list(layers)
        self.batch = batch
        self.dev = torch.device(device)
        self.p: List[Dict[str, torch.Tensor]] = []
        ws_bytes = 16
        for L, prm in zip(self.layers, params):
            d = {k: torch.from_numpy(np.ascontiguousarray(v)).to(self.dev) for k, v in prm.items()}
            if L.kind == "bconv":
                d["wp"] = B.bnn_pack_conv_weight(d["w"])
                ws_bytes = max(ws_bytes, B.conv2d_workspace_bytes((batch, L.cin, L.hw, L.hw), 3, 3, (1, 1), (1, 1)))
            elif L.kind == "bfc":
                d["wp"] = B.bnn_encode(d["w"])
            self.p.append(d)
        self.ws = torch.empty(ws_bytes, dtype=torch.uint8, device=self.dev)
        # activation buffers, allocated once
        self.buf: List[Dict[str, torch.Tensor]] = []
        for L in self.layers:
            b: Dict[str, torch.Tensor] = {}
            if L.kind == "conv_f32":
                b["y"] = torch.empty((batch, L.cout, L.hw, L.hw), dtype=torch.float32, device=self.dev)
            elif L.kind == "bconv":
                if L.pool:
                    b["acc"] = torch.empty((batch, L.cout, L.hw, L.hw), dtype=torch.int32, device=self.dev)
                    b["y"] = torch.empty((batch, L.cout, L.hw // 2, L.hw // 2), dtype=torch.float32, device=self.dev)
                else:
                    b["y"] = torch.empty((batch, L.cout, L.hw, L.hw), dtype=torch.float32, device=self.dev)
            elif L.kind == "bfc":
                b["xp"] = torch.empty((batch, B.packed_words(L.cin)), dtype=torch.int64, device=self.dev)
                b["y"] = torch.empty((batch, L.cout), dtype=torch.float32, device=self.dev)
            elif L.kind == "fc_f32":
                b["y"] = torch.empty((batch, L.cout), dtype=torch.float32, device=self.dev)
            self.buf.append(b)
        torch.cuda.synchronize(self.dev)

    def forward(self, x: torch.Tensor, keep: bool = False):
        h = x
        acts = []
        for L, p, b in zip(self.layers, self.p, self.buf):
            if L.kind == "conv_f32":
                h = B.bnn_conv2d_f32(h, p["w"], (1, 1), (1, 1), p["scale"], p["bias"], out=b["y"])
            elif L.kind == "bconv":
                if L.pool:
                    B.bnn_conv2d(h, p["wp"], L.cout, 3, 3, (1, 1), (1, 1), want_int=True, workspace=self.ws,
                                 out_i32=b["acc"])
                    _, h = B.bnn_maxpool2x2(b["acc"], p["scale"], p["bias"], want_int=False, out_f32=b["y"])
                else:
                    _, h = B.bnn_conv2d(h, p["wp"], L.cout, 3, 3, (1, 1), (1, 1), p["scale"], p["bias"],
                                        want_int=False, workspace=self.ws, out_f32=b["y"])
            elif L.kind == "bfc":
                xp = B.bnn_encode(h.view(self.batch, -1), b["xp"])
                _, h = B.bnn_xnor_gemm_epilogue(xp, p["wp"], L.cin, p["scale"], p["bias"], B.CH_COL, out_y=b["y"])
            elif L.kind == "fc_f32":
                h = B.bnn_fc_f32(h.view(self.batch, -1), p["w"], p["bias"], sign_input=True, out=b["y"])
            else:
                raise ValueError(L.kind)
            if keep:
                acts.append(h.clone())
        return (h, acts) if keep else h


class _ChainWeight:
    """A layer's packed filters and the copy of them in the order in which bnn_conv_chain multiplies.  The copy follows
    in-place changes of the filters by torch's version counter (inference tensors have none: it is renewed every time)."""

    def __init__(self, wp: torch.Tensor, cin: int):
        self.wp, self.cin, self.counted = wp, cin, not wp.is_inference()
        self.version = wp._version if self.counted else None
        self.wc = B.bnn_pack_conv_chain_weight(wp, cin)

    def refresh(self) -> None:
        if self.counted and self.wp._version == self.version:
            return
        self.version = self.wp._version if self.counted else None
        B.bnn_pack_conv_chain_weight(self.wp, self.cin, out=self.wc)


class _Chain:
    """Layers first .. last of a net through bnn_conv_chain, from the parameters that it holds when a pass is issued."""

    def __init__(self, first: int, last: int):
        self.first, self.last = first, last
        self.weights: Dict[int, _ChainWeight] = {}
        self.array = None

    def __getstate__(self):  # a copied net packs its own
        return {"first": self.first, "last": self.last, "weights": {}, "array": None}

    def host_array(self, net: "VggStackFused"):
        """Packed again, or built again, where a parameter has been changed or replaced since the last pass."""
        held = self.array.tensors if self.array is not None else None
        same = held is not None
        for k, i in enumerate(range(self.first, self.last + 1)):
            p = net.p[i]
            w = self.weights.get(i)
            if w is None or w.wp is not p["wp"]:  # w holds its tensor: the identity is not another's
                self.weights[i], same = _ChainWeight(p["wp"], net.layers[i].cin), False
            else:
                w.refresh()
            same = same and held[k][1] is p["scale"] and held[k][2] is p["bias"]
        if not same:
            self.array = _chain_array(net, {i: w.wc for i, w in self.weights.items()}, self.first, self.last)
        return self.array

    def run(self, net: "VggStackFused", x: torch.Tensor) -> torch.Tensor:
        return B.bnn_conv_chain(x, net.layers[self.first].cin, self.host_array(net), net.buf[self.last]["yp"])


def _chain_array(net: "VggStackFused", weights: Dict[int, torch.Tensor], first: int, last: int):
    return B.conv_chain_layers([(weights.get(i), net.p[i]["scale"], net.p[i]["bias"], net.layers[i].cout,
                                 2 if net.layers[i].pool else 0) for i in range(first, last + 1)])


class VggStackFused:
    """The same stack with activations kept packed between layers (1 bit per activation):
    real-valued first layer with binarized output, binarized convolutions whose GEMM store
    does max-pool + affine + sign + pack, and the binarized FC on the packed map with its
    weight re-ordered to the (h, w, c) bit order.  Same arithmetic, same results.

    A pass takes the parameters that p holds when it is issued.  Layers that go through bnn_conv_chain multiply a
    re-ordered copy of p[i]["wp"], which follows a replaced tensor and in-place changes that torch counts (copy_, indexing,
    other operators; in replay() of the tensors that were captured), not writes past torch's version counter (through
    .data, or by a raw address)."""

    def __init__(self, layers: Sequence, params: Sequence[Dict[str, np.ndarray]], batch: int, device="cuda:0"):
        self.layers = list(layers)
        self.batch = batch
        self.dev = torch.device(device)
        self.p: List[Dict[str, torch.Tensor]] = []
        self.buf: List[Dict[str, torch.Tensor]] = []
        hw_c = None  # (C, H, W) of the map entering the binarized FC
        for L, prm in zip(self.layers, params):
            d = {k: torch.from_numpy(np.ascontiguousarray(v)).to(self.dev) for k, v in prm.items()}
            b: Dict[str, torch.Tensor] = {}
            if L.kind == "conv_f32":
                b["yp"] = torch.empty((batch, L.hw, L.hw, B.packed_words(L.cout)), dtype=torch.int64, device=self.dev)
                hw_c = (L.cout, L.hw, L.hw)
            elif L.kind == "bconv":
                with torch.inference_mode(False):  # a version counter: see _ChainWeight
                    d["wp"] = B.bnn_pack_conv_weight(d["w"])
                o = L.hw // 2 if L.pool else L.hw
                b["yp"] = torch.empty((batch, o, o, B.packed_words(L.cout)), dtype=torch.int64, device=self.dev)
                hw_c = (L.cout, o, o)
            elif L.kind == "bfc":
                C, H, W = hw_c
                assert C * H * W == L.cin
                d["wp"] = B.bnn_pack_fc_weight_nhwc(d["w"], C, H, W)
                d["kbits"] = H * W * B.packed_words(C) * 64
                d["ktrue"] = L.cin
                b["y"] = torch.empty((batch, L.cout), dtype=torch.float32, device=self.dev)
            elif L.kind == "fc_f32":
                b["y"] = torch.empty((batch, L.cout), dtype=torch.float32, device=self.dev)
            self.p.append(d)
            self.buf.append(b)
        self._graph = None
        self._chain = self._find_chain()
        torch.cuda.synchronize(self.dev)

    def _find_chain(self):
        """The last consecutive binarized convolutions that go through bnn_conv_chain in one launch, as many of them as are
        expected to be faster than the layers one by one (bnn_conv_chain_pays), or None.
        Two maps of 128 channels of 32 x 32 do not fit LDS: the sixth convolution of the larger stack stays outside (its pass
        at batch 256 143 -> 121 us)."""
        conv = [i for i, L in enumerate(self.layers) if L.kind == "bconv"]
        if not conv or conv != list(range(conv[0], conv[-1] + 1)):
            return None
        for first in conv:
            L0 = self.layers[first]
            if first > 0 and B.bnn_conv_chain_pays(self.batch, L0.cin, L0.hw, L0.hw, _chain_array(self, {}, first, conv[-1])):
                chain = _Chain(first, conv[-1])
                chain.host_array(self)
                return chain
        return None

    def capture(self, x: torch.Tensor) -> None:
        """Record one forward pass reading x (its storage, not its present contents) into a HIP
        graph.  Every buffer of the pass is preallocated and the library neither allocates nor
        synchronises, so the graph holds exactly the pass's kernel launches; replay() re-issues
        them with one submission, which is what matters at batch sizes where a pass is shorter
        than its eight launches take to submit."""
        side = torch.cuda.Stream(device=self.dev)  # default priority
        side.wait_stream(torch.cuda.current_stream(self.dev))
        with torch.cuda.stream(side):
            self.forward(x)  # every code path has run once before capture
        torch.cuda.current_stream(self.dev).wait_stream(side)
        torch.cuda.synchronize(self.dev)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            self._graph_out = self.forward(x)
        self._graph = g
        # what the graph reads: its tensors live as long as it does, and replay() keeps the copies in step with the filters
        self._graph_weights = list(self._chain.weights.values()) if self._chain else []
        self._graph_array = self._chain.array if self._chain else None

    def replay(self) -> torch.Tensor:
        """Re-run the captured pass on the current contents of the captured input."""
        if self._graph is None:
            raise RuntimeError("capture() first")
        for w in self._graph_weights:
            w.refresh()
        self._graph.replay()
        return self._graph_out

    def forward(self, x: torch.Tensor, keep: bool = False):
        h = x
        acts = []
        chain = None if keep else self._chain  # the maps inside the chain never reach memory
        for i, (L, p, b) in enumerate(zip(self.layers, self.p, self.buf)):
            if chain and chain.first <= i <= chain.last:
                if i == chain.first:
                    h = chain.run(self, h)
                continue
            if L.kind == "conv_f32":
                h = B.bnn_conv2d_f32_sign(h, p["w"], p["scale"], p["bias"], (1, 1), (1, 1), out=b["yp"])
            elif L.kind == "bconv":
                h = B.bnn_conv2d_packed(h, p["wp"], L.cin, L.cout, 3, 3, (1, 1), (1, 1), pool=2 if L.pool else 0,
                                        scale=p["scale"], bias=p["bias"], out="packed", out_buf=b["yp"])
            elif L.kind == "bfc":
                # pad bits are 0 in both operands, so the GEMM runs over whole words and the
                # formula takes the true K through the epilogue entry point's K argument
                rows = h.view(self.batch, -1)
                assert rows.shape[1] * 64 == p["kbits"] == p["ktrue"], "channel counts here are multiples of 64"
                _, h = B.bnn_xnor_gemm_epilogue(rows, p["wp"], p["ktrue"], p["scale"], p["bias"], B.CH_COL,
                                                out_y=b["y"])
            elif L.kind == "fc_f32":
                h = B.bnn_fc_f32(h.view(self.batch, -1), p["w"], p["bias"], sign_input=True, out=b["y"])
            else:
                raise ValueError(L.kind)
            if keep:
                acts.append(h.clone())
        return (h, acts) if keep else h

    def conv_launches(self):
        """One closure per launch of binarized convolutions (a layer's, or the chain's) that re-issues exactly that launch
        on the buffers the last forward() left behind (for timing a launch in isolation)."""
        out = []
        prev = None
        for i, (L, p, b) in enumerate(zip(self.layers, self.p, self.buf)):
            if self._chain and i == self._chain.first:
                out.append(lambda: self._chain.run(self, self.buf[self._chain.first - 1]["yp"]))
                break
            if L.kind == "bconv":
                src = prev

                def call(L=L, p=p, b=b, src=src):
                    B.bnn_conv2d_packed(src, p["wp"], L.cin, L.cout, 3, 3, (1, 1), (1, 1), pool=2 if L.pool else 0,
                                        scale=p["scale"], bias=p["bias"], out="packed", out_buf=b["yp"])
                out.append(call)
            prev = b.get("yp", None)
        return out


class SplitBatch:
    """The fused stack on `parts` equal slices of the batch, each on its own HIP stream (default
    priority).  Images are independent, so the slices need no exchange; while one slice drains
    the tail of a kernel the other's next kernel fills the idle compute units."""

    def __init__(self, layers, params, batch: int, parts: int = 2, device="cuda:0"):
        assert batch % parts == 0
        self.parts = parts
        self.bs = batch // parts
        self.nets = [VggStackFused(layers, params, batch=self.bs, device=device) for _ in range(parts)]
        self.streams = [torch.cuda.Stream(device=device) for _ in range(parts)]

    def fork(self):
        """Make the slice streams wait for what has been enqueued on the current stream."""
        main = torch.cuda.current_stream()
        for st in self.streams:
            st.wait_stream(main)

    def join(self):
        """Make the current stream wait for everything enqueued on the slice streams."""
        main = torch.cuda.current_stream()
        for st in self.streams:
            main.wait_stream(st)

    def forward(self, x: torch.Tensor, sync: bool = True):
        """sync=False only enqueues the slices (successive batches then overlap freely; the caller
        forks before the first and joins after the last)."""
        if sync:
            self.fork()
        outs = []
        for i, (net, st) in enumerate(zip(self.nets, self.streams)):
            with torch.cuda.stream(st):
                outs.append(net.forward(x[i * self.bs:(i + 1) * self.bs]))
        if sync:
            self.join()
        return outs
