"""Work that programs using this library have it do, as measurable cases.

A case is a pipeline (an OpenVX-style graph of the library's nodes, or calls
of its immediate-mode operators), an image size, a number of frames and the
border rule.  Images are synthetic camera-like frames: smooth shading, flat
rectangles with sharp edges, sensor noise.

Every output but two kinds holds whole numbers (pixels, counts, exact sums);
the F32 corner response and the F32 mean and standard deviation are the
computed ones, and ``exact`` gives those in 64 bits.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2008_11476_amd as hvx

U8, S16, F32, UYVY = hvx.HVX_DF_U8, hvx.HVX_DF_S16, hvx.HVX_DF_F32, hvx.HVX_DF_UYVY
BORDERS = {"replicate": hvx.HVX_BORDER_REPLICATE, "constant": hvx.HVX_BORDER_CONSTANT,
           "mirror": hvx.HVX_BORDER_MIRROR}
HARRIS_K = 0.04


# ---- the pipelines: nodes between an input image and the output images -------

def _edge(g, a, outs, border):
    v = [hvx.hvx_image_create_virtual(g) for _ in range(4)]
    nodes = [hvx.hvx_gaussian3x3_node(g, a, v[0]), hvx.hvx_sobel3x3_node(g, v[0], v[1], v[2])]
    hvx.hvx_magnitude_node(g, v[1], v[2], v[3])
    hvx.hvx_threshold_node(g, v[3], 100.0, 255, 0, outs[0])
    if len(outs) > 1:
        hvx.hvx_phase_node(g, v[1], v[2], outs[1])
    return nodes


def _structure_tensor(g, a):
    """Sobel, the three products and their 5x5 box sums."""
    v = [hvx.hvx_image_create_virtual(g) for _ in range(8)]
    nodes = [hvx.hvx_sobel3x3_node(g, a, v[0], v[1])]
    for (p, q, o) in ((0, 0, 2), (1, 1, 3), (0, 1, 4)):
        hvx.hvx_multiply_f32_node(g, v[p], v[q], v[o])
        nodes.append(hvx.hvx_box5x5_f32_node(g, v[o], v[o + 3]))
    return v[5:8], nodes


def _corner(g, a, outs, border):
    s, nodes = _structure_tensor(g, a)
    r = hvx.hvx_image_create_virtual(g)
    hvx.hvx_harris_response_node(g, s[0], s[1], s[2], HARRIS_K, r)
    hvx.hvx_threshold_node(g, r, 1e6, 255, 0, outs[0])
    return nodes


def _response(g, a, outs, border):
    s, nodes = _structure_tensor(g, a)
    hvx.hvx_harris_response_node(g, s[0], s[1], s[2], HARRIS_K, outs[0])
    return nodes


def _tomasi(g, a, outs, border):
    s, nodes = _structure_tensor(g, a)
    r = hvx.hvx_image_create_virtual(g)
    hvx.hvx_custom_point_node(g, "(a + b) / 2 - sqrt((a - b) * (a - b) / 4 + c * c)", s, F32, r)
    hvx.hvx_threshold_node(g, r, 2e5, 255, 0, outs[0])
    return nodes


def _gauss5(g, a, outs, border):
    return [hvx.hvx_gaussian5x5_node(g, a, outs[0])]


def _uyvy_gauss5(g, a, outs, border):
    y = hvx.hvx_image_create_virtual(g)
    hvx.hvx_channel_extract_node(g, a, hvx.HVX_CHANNEL_Y, y)
    return [hvx.hvx_gaussian5x5_node(g, y, outs[0])]


def _unsharp(g, a, outs, border):
    v = [hvx.hvx_image_create_virtual(g) for _ in range(3)]
    nodes = [hvx.hvx_gaussian3x3_node(g, a, v[0])]
    hvx.hvx_custom_point_node(g, "a - b", [a, v[0]], S16, v[1])
    hvx.hvx_custom_point_node(g, "a * 3 / 2", [v[1]], S16, v[2])
    hvx.hvx_custom_point_node(g, "a + b", [a, v[2]], U8, outs[0])
    return nodes


FCHAIN_MASKS = (([[i * j for i in (1, 4, 6, 4, 1)] for j in (1, 4, 6, 4, 1)], 256),
                ([[0, -1, 0], [-1, 5, -1], [0, -1, 0]], 1),
                ([[1] * 5] * 5, 32))


def _fchain(g, a, outs, border):
    v = [hvx.hvx_image_create_virtual(g, 0, 0, U8) for _ in range(2)]
    chain = [a, v[0], v[1], outs[0]]
    return [hvx.hvx_convolve_node(g, chain[k], _mask(k), chain[k + 1]) for k in range(3)]


def _thin(g, a, outs, border):
    v = [hvx.hvx_image_create_virtual(g) for _ in range(4)]
    nodes = [hvx.hvx_median3x3_node(g, a, v[0]), hvx.hvx_sobel3x3_node(g, v[0], v[1], v[2])]
    hvx.hvx_magnitude_node(g, v[1], v[2], v[3])
    return nodes + [hvx.hvx_non_max_suppression_node(g, v[3], 3, outs[0])]


# name: (builder, input format, output formats, bytes and operations per pixel)
GRAPHS = {
    "edge": (_edge, U8, (U8,), 2, 25),
    "edge_phase": (_edge, U8, (U8, U8), 3, 40),
    "corner": (_corner, U8, (U8,), 2, 45),
    "response": (_response, U8, (F32,), 5, 44),
    "tomasi": (_tomasi, U8, (U8,), 2, 48),
    "gauss5": (_gauss5, U8, (U8,), 2, 18),
    "uyvy_gauss5": (_uyvy_gauss5, UYVY, (U8,), 3, 18),
    "unsharp": (_unsharp, U8, (U8,), 2, 15),
    "fchain": (_fchain, U8, (U8,), 2, 40),
    "thin": (_thin, U8, (S16,), 3, 45),
}

_ctx = None
_convs = {}


def _context():
    global _ctx
    if _ctx is None:
        _ctx = hvx.hvx_context_create(0)
    return _ctx


def _mask(k):
    if k not in _convs:
        coeffs, scale = FCHAIN_MASKS[k]
        _convs[k] = hvx.hvx_convolution_create(_context(), coeffs, scale)
    return _convs[k]


# ---- the cases ----------------------------------------------------------------

def listed():
    return [
        # a camera frame analysed as it arrives: one small frame, one launch; latency counts
        dict(name="edge_phase_vga", kind="frame", graph="edge_phase", w=640, h=480, border="replicate"),
        # the throughput workload: edge map and gradient direction of 64 4K frames, one batch
        dict(name="edge_phase_4k_batch64", kind="batch", graph="edge_phase", w=3840, h=2160, n=64,
             border="replicate"),
        # an image collection of mixed odd sizes through mixed detectors, one batch
        dict(name="mixed_batch64", kind="mixed", w=4096, h=2160, n=64, shapes=0),
        # video frames in their camera format: luma and blur of a short 1080p clip
        dict(name="uyvy_gauss5_1080p_batch32", kind="batch", graph="uyvy_gauss5", w=1920, h=1080, n=32,
             border="constant"),
        # sharpening one 4K photograph, with user point kernels
        dict(name="unsharp_4k", kind="frame", graph="unsharp", w=3840, h=2160, border="replicate"),
        # corner features with a user response over 32 4K frames
        dict(name="tomasi_4k_batch32", kind="batch", graph="tomasi", w=3840, h=2160, n=32, border="replicate"),
        # a chain of user masks on one 4K frame
        dict(name="fchain_4k", kind="frame", graph="fchain", w=3840, h=2160, border="replicate"),
        # the F32 corner response of an image with an odd size, for a later stage of the program's own
        dict(name="response_odd", kind="frame", graph="response", w=1021, h=1019, border="constant"),
        # thin edges of a denoised 1080p frame: median, gradient magnitude, non-maximum suppression on S16
        dict(name="thin_1080p", kind="frame", graph="thin", w=1920, h=1080, border="mirror"),
        # exposure statistics of a smoothed 4K frame: histogram, mean and standard deviation in one graph
        dict(name="smooth_stats_4k", kind="stats", w=3840, h=2160, border="replicate"),
        # a 16k scan equalised, with its extremes: the immediate-mode global operators
        dict(name="equalize_16k", kind="global", w=16384, h=16384),
        # a burst of mixed requests on resident frames through the server
        dict(name="serve_burst24", kind="serve", n=24, shapes=0),
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("frame", "frame", "frame", "batch", "batch", "batch", "mixed", "stats", "global", "serve"))
    w, h = _log_size(rng, 320, 4096), _log_size(rng, 240, 2160)
    border = rng.choice(tuple(BORDERS))
    if kind == "stats":
        return dict(kind=kind, w=w, h=h, border=border)
    if kind == "global":
        return dict(kind=kind, w=_log_size(rng, 320, 16384), h=_log_size(rng, 240, 16384))
    if kind == "mixed":
        return dict(kind=kind, w=4096, h=2160, n=_log_size(rng, 2, 64), shapes=rng.randrange(1, 1 << 20))
    if kind == "serve":
        return dict(kind=kind, n=rng.randrange(4, 25), shapes=rng.randrange(1, 1 << 20))
    graph = rng.choice(tuple(GRAPHS))
    if graph == "uyvy_gauss5":
        w += w % 2
    c = dict(kind=kind, graph=graph, w=w, h=h, border=border)
    if kind == "batch":
        most = 32 * 3840 * 2160 * 2 // GRAPHS[graph][3]  # at most the bytes of 32 4K frames in and out
        c["n"] = _log_size(rng, 2, max(2, min(64, most // (w * h))))
    return c


MIXED_GRAPHS = ("edge", "corner", "gauss5")
SERVE_GRAPHS = ("edge", "corner", "uyvy_gauss5")
SERVE_SIZES = ((640, 480), (1280, 720), (1920, 1080), (3840, 2160))


def _shapes(case):
    """(graph, width, height) of each image of a mixed batch or of each request."""
    rng = random.Random(case["shapes"])
    if case["kind"] == "serve":
        return [(rng.choice(SERVE_GRAPHS),) + rng.choice(SERVE_SIZES) for _ in range(case["n"])]
    return [(rng.choice(MIXED_GRAPHS), rng.randint(320, case["w"]), rng.randint(240, case["h"]))
            for _ in range(case["n"])]


def work(case):
    kind = case["kind"]
    if kind in ("mixed", "serve"):
        per = [(GRAPHS[g][3] * w * h, GRAPHS[g][4] * w * h) for (g, w, h) in _shapes(case)]
        return {"bytes": sum(b for b, _ in per), "flops": sum(f for _, f in per)}
    px = case["w"] * case["h"] * case.get("n", 1)
    if kind == "stats":
        return {"bytes": px, "flops": 13 * px}
    if kind == "global":
        return {"bytes": 2 * px, "flops": 6 * px}
    return {"bytes": GRAPHS[case["graph"]][3] * px, "flops": GRAPHS[case["graph"]][4] * px}


# ---- inputs ---------------------------------------------------------------------

def _frame(w, h, gen):
    """A camera-like U8 frame: smooth shading, 12 flat rectangles, noise."""
    dev = "cuda"
    coarse = torch.rand((1, 1, 7, 9), generator=gen, device=dev) * 160 + 40
    img = torch.nn.functional.interpolate(coarse, size=(h, w), mode="bilinear", align_corners=True)[0, 0]
    img = img + torch.randn((h, w), generator=gen, device=dev) * 6
    u = torch.rand((12, 5), generator=gen, device=dev).cpu().tolist()
    for (x, y, rw, rh, level) in u:
        x0, y0 = int(x * w), int(y * h)
        img[y0:y0 + 1 + int(rh * h / 4), x0:x0 + 1 + int(rw * w / 4)] = level * 255
    return img.round().clamp(0, 255).to(torch.uint8)


def _input(df, w, h, gen):
    buf, view = hvx.alloc_image(h, w, df)
    if df == UYVY:
        view[:, 1::2] = _frame(w, h, gen)
        view[:, 0::2] = torch.randint(96, 160, (h, w), generator=gen, device="cuda", dtype=torch.uint8)
    else:
        view.copy_(_frame(w, h, gen))
    return view


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return gen


class _State:
    """What a program keeps: frames, output buffers, images, graphs, a batch
    or a server.  Released with the state."""

    def __init__(self):
        self.inputs, self.outputs, self.images, self.graphs, self.buffers = [], [], [], [], []
        self.batch = self.server = None
        self.extra = {}

    def image(self, view, df):
        w = view.shape[1] // 2 if df == UYVY else view.shape[1]
        im = hvx.image_from_tensor(_context(), view, df, w=w)
        self.images.append(im)
        return im

    def graph(self, name, w, h, border, gen, dst=None):
        """A verified graph over a new frame, writing to `dst` (new images by default)."""
        build, idf, odfs = GRAPHS[name][:3]
        src = _input(idf, w, h, gen)
        if dst is None:
            dst = [hvx.alloc_image(h, w, df)[1] for df in odfs]
            self.outputs.append(dst)
        g = hvx.hvx_graph_create(_context())
        a = self.image(src, idf)
        o = [self.image(d, df) for d, df in zip(dst, odfs)]
        for node in build(g, a, o, border):
            hvx.hvx_node_set_border(node, BORDERS[border], 0)
        hvx.hvx_graph_verify(g, ctx=_context())
        self.inputs.append(src)
        self.graphs.append(g)
        return g, a, o

    def __del__(self):
        try:
            torch.cuda.synchronize()
            if self.server is not None:
                hvx.hvx_release_server(self.server)
            if self.batch is not None:
                hvx.hvx_release_batch(self.batch)
            for g in self.graphs:
                hvx.hvx_release_graph(g)
            for im in self.images:
                hvx.hvx_release_image(im)
            for b in self.buffers:
                hvx.hvx_release_buffer(b)
        except Exception:  # the interpreter is going down
            pass


def prepare(case, seed):
    gen = _generator(seed)
    s = _State()
    kind = case["kind"]
    ctx = _context()
    if kind == "frame":
        s.graph(case["graph"], case["w"], case["h"], case["border"], gen)
    elif kind == "batch":
        # the frames' outputs lie one after another in one buffer per output
        n, w, h = case["n"], case["w"], case["h"]
        s.outputs = [hvx.alloc_image(n * h, w, df)[1] for df in GRAPHS[case["graph"]][2]]
        for i in range(n):
            s.graph(case["graph"], w, h, case["border"], gen, [o[i * h:(i + 1) * h] for o in s.outputs])
        s.batch = hvx.hvx_batch_create(ctx, s.graphs)
    elif kind == "mixed":
        for (name, w, h) in _shapes(case):
            s.graph(name, w, h, "replicate", gen)
        s.batch = hvx.hvx_batch_create(ctx, s.graphs)
    elif kind == "serve":
        s.extra["requests"] = []
        for (name, w, h) in _shapes(case):
            g, a, o = s.graph(name, w, h, "replicate", gen)
            bind = [(a,) + hvx.tensor_args(s.inputs[-1]), (o[0],) + hvx.tensor_args(s.outputs[-1][0])]
            s.extra["requests"].append((g, bind))
        s.server = hvx.hvx_server_create(ctx, hvx.HVX_SERVER_CONTINUOUS, 512 << 20, 16, 2)
    elif kind == "stats":
        src = _input(U8, case["w"], case["h"], gen)
        counts = torch.zeros(256, dtype=torch.int32, device="cuda")
        stat = torch.zeros(3, dtype=torch.int64, device="cuda")
        g = hvx.hvx_graph_create(ctx)
        v = hvx.hvx_image_create_virtual(g)
        node = hvx.hvx_gaussian3x3_node(g, s.image(src, U8), v)
        hvx.hvx_node_set_border(node, BORDERS[case["border"]], 0)
        s.buffers = [hvx.hvx_buffer_from_ptr(ctx, counts.data_ptr(), 1024),
                     hvx.hvx_buffer_from_ptr(ctx, stat.data_ptr(), 24)]
        hvx.hvx_histogram_node(g, v, 256, 0, 256, s.buffers[0])
        hvx.hvx_mean_std_dev_node(g, v, s.buffers[1])
        hvx.hvx_graph_verify(g, ctx=ctx)
        s.inputs, s.graphs = [src], [g]
        s.outputs = [[counts, stat[:2], stat[2:].view(torch.float32)]]
    else:  # global
        src = _input(U8, case["w"], case["h"], gen)
        dst = hvx.alloc_image(case["h"], case["w"], U8)[1]
        s.extra["in"], s.extra["out"] = s.image(src, U8), s.image(dst, U8)
        s.extra["table"] = torch.zeros(160, dtype=torch.int64, device="cuda")
        s.extra["result"] = torch.zeros(1032, dtype=torch.int32, device="cuda")
        s.inputs = [src]
        s.outputs = [[dst, s.extra["result"][:4]]]
    torch.cuda.synchronize()
    return s


# ---- one pass ---------------------------------------------------------------------

def run(state):
    stream = torch.cuda.current_stream().cuda_stream
    if state.batch is not None:
        hvx.hvx_batch_schedule(state.batch, stream)
    elif state.server is not None:
        for tag, (g, bind) in enumerate(state.extra["requests"]):
            hvx.hvx_server_submit_bound(state.server, g, bind, hvx.HVX_MEMORY_DEVICE, tag)
        hvx.hvx_server_drain(state.server)
        done = hvx.hvx_server_poll(state.server)
        if any(status for (_, status, _) in done):
            raise RuntimeError("a request failed")
    elif state.graphs:
        hvx.hvx_graph_schedule(state.graphs[0], stream)
    else:
        e = state.extra
        hvx.hvx_min_max_count(_context(), e["in"], e["result"].data_ptr(), stream)
        hvx.hvx_equalize_hist(_context(), e["in"], e["out"], e["table"].data_ptr(), stream)
    return state.outputs


# ---- the computed numbers in 64 bits -------------------------------------------------

def _pad(img, r, border):
    """`img` (float64, H x W) with r pixels of its border rule around it."""
    if border == "constant":
        return torch.nn.functional.pad(img, (r, r, r, r))

    def index(n):
        i = torch.arange(-r, n + r, device=img.device)
        if border == "mirror" and n > 1:
            i = i.remainder(2 * n - 2)
            return torch.minimum(i, 2 * n - 2 - i)
        return i.clamp(0, n - 1)

    return img[index(img.shape[0])][:, index(img.shape[1])]


def _filter(img, col, row, border):
    """The separable correlation with weights col (vertical) and row."""
    r = len(row) // 2
    p = _pad(img, r, border)
    h, w = img.shape
    t = sum(c * p[i:i + h] for i, c in enumerate(col))
    return sum(c * t[:, i:i + w] for i, c in enumerate(row))


def _response_exact(img, border):
    a = img.double()
    gx, gy = _filter(a, (1, 2, 1), (-1, 0, 1), border), _filter(a, (-1, 0, 1), (1, 2, 1), border)
    ones = (1,) * 5
    sxx, syy, sxy = (_filter(p, ones, ones, border) for p in (gx * gx, gy * gy, gx * gy))
    # the node takes k as an F32 number
    return sxx * syy - sxy * sxy - float(np.float32(HARRIS_K)) * (sxx + syy) ** 2


def exact(case, seed):
    kind = case["kind"]
    if kind == "stats":
        img = _input(U8, case["w"], case["h"], _generator(seed))
        g = torch.floor(_filter(img.double(), (1, 2, 1), (1, 2, 1), case["border"]) / 16)
        # _filter pads rows and columns alike, so the corners follow the rule too
        mean, var = g.mean(), g.var(unbiased=False)
        return [[None, None, torch.stack([mean, var.sqrt()])]]
    if case.get("graph") == "response":
        gen = _generator(seed)
        r = [_response_exact(_input(U8, case["w"], case["h"], gen), case["border"]) for _ in range(case.get("n", 1))]
        return [torch.cat(r)] if kind == "batch" else [r]
    return None  # whole numbers only
