"""Performance cases: the work a user of this library has it do, through the
public entry points of paper_1907_03739_amd (binding and network).

Kinds of case, each with the sizes the repository's workloads and tests use:

  layer   inference of one PVConv layer, one call (pvconv_forward): the
          part-segmentation layer, a network's inner layer, the large clustered
          cloud, the small fp32 layer, the narrow (compact model) widths, grids
          whose faces cut the kernels' bricks, point counts of no round number
  train   forward and backward of one PVConv layer from the separate entry
          points, as a training program that keeps the activations calls them:
          gradients of the features and of the convolutions' weights
  sa      one PointNet++ set abstraction: sampling, ball query, grouping,
          shared MLP, maximum over the neighbours
  fp      one PointNet++ feature propagation: three nearest neighbours,
          interpolation beside the skip features, shared MLP
  head    the point-only tail of the part-segmentation network: wide shared
          MLPs, the global maximum, the head on every stage's features
  pvcnn   a whole segmentation network (DeviceNetwork), to its logits
  pvcnn2  a whole PVCNN++ (DevicePVCNN2), to its logits

Inputs are synthetic: points on the surfaces of random boxes and spheres
(shapes, rooms) or clusters, standard normal features, Kaiming weights.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

DEV = "cuda"
BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64
SLOPE = 0.1


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _layer(name, B, N, cin, cout, R, convs, cloud, compute="bf16", feat="f32", out="f32",
           devox="trilinear"):
    c = dict(kind="layer", B=B, N=N, cin=cin, cout=cout, R=R, convs=convs, cloud=cloud,
             compute=compute, feat=feat, out=out, devox=devox)
    return dict(c, name=name) if name else c


def _train(name, B, N, cin, cout, R, cloud):
    c = dict(kind="train", B=B, N=N, cin=cin, cout=cout, R=R, cloud=cloud)
    return dict(c, name=name) if name else c


def _sa(name, B, N, M, cin, w1, w2, w3, radius, nsample=32):
    c = dict(kind="sa", B=B, N=N, M=M, cin=cin, w1=w1, w2=w2, w3=w3, radius=radius,
             nsample=nsample)
    return dict(c, name=name) if name else c


def _fp(name, B, N, M, cdeep, cskip, width, layers):
    c = dict(kind="fp", B=B, N=N, M=M, cdeep=cdeep, cskip=cskip, width=width, layers=layers)
    return dict(c, name=name) if name else c


def _whole(kind, name, B, N, width):
    c = dict(kind=kind, B=B, N=N, width=width)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small fp32 layer on one cloud: launches and latency
        _layer("layer_f32_small", 1, 1024, 16, 32, 8, 1, "cube", compute="f32"),
        # the part-segmentation layer, the benchmark's own: inference of a batch
        _layer("layer_part", 16, 2048, 64, 128, 32, 2, "shape"),
        # one large cloud with most points in a few voxels
        _layer("layer_cluster", 1, 65536, 64, 64, 64, 2, "cluster"),
        # an inner layer of the scene network: bf16 rows in and out, R = 16
        _layer("layer_inner", 8, 4096, 64, 128, 16, 2, "room", feat="bf16", out="bf16"),
        # a compact model's layer on odd sizes: widths of 24 and 40, R = 20
        _layer("layer_ragged", 3, 1777, 24, 40, 20, 2, "room"),
        # a training step of the part-segmentation layer
        _train("train_part", 8, 2048, 64, 128, 32, "shape"),
        # the same of a small grid, odd number of clouds and points
        _train("train_small", 3, 1500, 32, 64, 16, "room"),
        # the scene PVCNN++'s first set abstraction (8192 -> 1024 centres)
        _sa("sa_first", 4, 8192, 1024, 32, 32, 32, 64, 0.2),
        # its last feature propagation (1024 -> 8192 points)
        _fp("fp_last", 4, 8192, 1024, 128, 32, 128, 3),
        # the part-segmentation network's tail
        _whole("head", "head_part", 8, 2048, 1.0),
        # whole networks: the part-segmentation PVCNN, the scene PVCNN++
        _whole("pvcnn", "pvcnn_part", 8, 2048, 1.0),
        _whole("pvcnn2", "pvcnn2_scene", 4, 8192, 1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer"] * 5 + ["train"] * 2 + ["sa"] * 2 + ["fp"] * 2 +
                      ["head", "pvcnn", "pvcnn2"])
    if kind == "layer":
        while True:
            if rng.random() < 0.15:  # fp32: small layers
                B, N = rng.randint(1, 4), _log_int(rng, 200, 2048)
                return _layer(None, B, N, rng.choice([3, 9, 16, 20, 32]),
                              rng.choice([8, 16, 30, 32]), rng.randint(5, 14), rng.randint(1, 2),
                              rng.choice(["cube", "shape"]), compute="f32")
            big = rng.random() < 0.2
            B = 1 if big else _log_int(rng, 1, 16)
            N = _log_int(rng, 8192, 65536) if big else _log_int(rng, 300, 4096)
            cin = rng.choice([3, 9, 16, 24, 32, 48, 64, 64, 96, 128])
            cout = rng.choice([16, 24, 40, 32, 64, 64, 96, 128])
            R = rng.randint(28, 64) if big else rng.randint(8, 36)
            convs = rng.choice([1, 2, 2, 2, 3])
            flops = 54.0 * B * R ** 3 * cout * (cin + (convs - 1) * cout)
            if flops <= 7.0e11:
                break
        return _layer(None, B, N, cin, cout, R, convs,
                      rng.choice(["cluster", "room", "shape"]) if big else
                      rng.choice(["shape", "shape", "room", "cube"]),
                      feat=rng.choice(["f32", "bf16"]) if cin >= 16 else "f32",
                      out=rng.choice(["f32", "bf16"]),
                      devox=rng.choice(["trilinear"] * 5 + ["nearest"]))
    if kind == "train":
        while True:
            B, N, R = _log_int(rng, 1, 12), _log_int(rng, 300, 4096), rng.randint(8, 34)
            cin, cout = rng.choice([32, 64, 96, 128]), rng.choice([64, 128])
            if 54.0 * B * R ** 3 * cout * (cin + cout) <= 3.4e11:
                return _train(None, B, N, cin, cout, R, rng.choice(["shape", "room", "cube"]))
    if kind == "sa":
        N = _log_int(rng, 128, 8192)
        M = max(1, int(N / rng.uniform(4.0, 8.5)))
        w = rng.choice([16, 32, 64])
        return _sa(None, rng.randint(1, 8 if N < 4096 else 4), N, M, rng.choice([9, 32, 61, 64]),
                   w, w, 2 * w, round(rng.uniform(0.2, 0.8), 2), rng.choice([16, 32, 32]))
    if kind == "fp":
        N = _log_int(rng, 64, 8192)
        return _fp(None, rng.randint(1, 4), N, max(3, int(N / rng.uniform(4.0, 8.5))),
                   rng.choice([64, 128, 256]), rng.choice([9, 32, 64, 128]),
                   rng.choice([64, 128, 256]), rng.randint(1, 3))
    width = rng.choice([0.25, 0.5, 0.75, 1.0])
    if kind == "pvcnn2":
        return _whole(kind, None, rng.randint(1, 4), _log_int(rng, 1200, 8192), width)
    return _whole(kind, None, rng.randint(1, 8), _log_int(rng, 600, 2048), width)


# --------------------------------------------------------------------------
# inputs (numpy, from the seed alone)
# --------------------------------------------------------------------------
def _box_points(rng, n, lo, hi):
    """n points uniform on the faces of the box [lo, hi]."""
    ext = hi - lo
    area = np.array([ext[1] * ext[2], ext[0] * ext[2], ext[0] * ext[1]])
    ax = rng.choice(3, size=n, p=area / area.sum())
    p = lo + rng.random((n, 3)) * ext
    side = rng.integers(0, 2, size=n)
    rows = np.arange(n)
    p[rows, ax] = np.where(side == 0, lo[ax], hi[ax])
    return p


def _cloud(rng, kind, B, N):
    """[B][N][3] float32: 'cube' uniform in a cube; 'shape' one to four boxes and
    spheres with jitter; 'room' a room's walls with boxes on its floor (metres);
    'cluster' four fifths of the points in sixteen tight clusters."""
    out = np.empty((B, N, 3), np.float32)
    for b in range(B):
        if kind == "cube":
            p = rng.uniform(-1.0, 1.0, size=(N, 3))
        elif kind == "shape":
            parts, k = [], int(rng.integers(1, 5))
            for n in rng.multinomial(N, np.full(k, 1.0 / k)):
                q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
                if rng.random() < 0.4:
                    v = rng.normal(size=(n, 3))
                    s = v / np.linalg.norm(v, axis=1, keepdims=True) * rng.uniform(0.2, 0.6)
                else:
                    h = rng.uniform(0.1, 0.5, size=3)
                    s = _box_points(rng, n, -h, h)
                parts.append(s @ q.T + rng.uniform(-0.5, 0.5, size=3))
            p = np.concatenate(parts) + rng.normal(scale=0.01, size=(N, 3))
        elif kind == "room":
            room = np.array([rng.uniform(3, 8), rng.uniform(3, 8), 3.0])
            boxes = [(np.zeros(3), room)]
            for _ in range(int(rng.integers(5, 16))):
                s = rng.uniform(0.3, 1.5, size=3)
                lo = np.array([rng.uniform(0, room[0] - s[0]), rng.uniform(0, room[1] - s[1]), 0])
                boxes.append((lo, lo + s))
            area = np.array([2 * (e[0] * e[1] + e[1] * e[2] + e[0] * e[2])
                             for e in (hi - lo for lo, hi in boxes)])
            n = rng.multinomial(N, area / area.sum())
            p = np.concatenate([_box_points(rng, int(k), lo, hi) for k, (lo, hi) in zip(n, boxes)])
        else:
            n = int(round(0.8 * N))
            which = rng.integers(0, 16, size=n)
            mean = rng.uniform(-0.8, 0.8, size=(16, 3))
            sig = np.exp(rng.uniform(math.log(0.01), math.log(0.06), size=(16, 3)))
            p = np.concatenate([rng.normal(size=(n, 3)) * sig[which] + mean[which],
                                rng.uniform(-1.0, 1.0, size=(N - n, 3))])
        out[b] = p[rng.permutation(N)]
    return out


def _normal(rng, shape, scale=1.0):
    return torch.from_numpy(rng.standard_normal(size=shape, dtype=np.float32) * np.float32(scale))


def _bn(rng, C):
    f = lambda a: torch.from_numpy(a.astype(np.float32))  # noqa: E731
    return SimpleNamespace(gamma=f(rng.uniform(0.5, 1.5, C)), beta=f(rng.uniform(-0.5, 0.5, C)),
                           mean=f(rng.normal(0, 0.5, C)), var=f(rng.uniform(0.5, 2.0, C)),
                           eps=1e-5)


def _weight(rng, shape, fan_in, bf16=True):
    """Kaiming normal; for the bf16 path already a bf16 value."""
    w = _normal(rng, shape, math.sqrt(2.0 / fan_in))
    return w.to(BF16).float() if bf16 else w


def _linear(rng, cin, cout, final=False):
    w = _weight(rng, (cout, cin), cin)
    if final:
        b = torch.from_numpy(rng.uniform(-0.1, 0.1, cout).astype(np.float32))
        return SimpleNamespace(w=w, b=b, bn=None, relu=False)
    return SimpleNamespace(w=w, b=None, bn=_bn(rng, cout), relu=True)


def _pvconv(rng, cin, cout, R, convs, bf16=True, devox="trilinear"):
    ws, c = [], cin
    for _ in range(convs):
        ws.append(_weight(rng, (cout, 3, 3, 3, c), 27 * c, bf16))
        c = cout
    return SimpleNamespace(cin=cin, cout=cout, R=R, n_convs=convs, conv_w=ws,
                           conv_bn=[_bn(rng, cout) for _ in range(convs)],
                           mlp_w=_weight(rng, (cout, cin), cin, bf16), mlp_b=None,
                           mlp_bn=_bn(rng, cout), slope=SLOPE, devox=devox)


def _scale(width):
    return lambda c: max(1, int(round(c * width)))


def _pvcnn_params(rng, width):
    """The part-segmentation PVCNN: blocks, point MLPs, head."""
    w = _scale(width)
    blocks, c = [], 3
    for cout, R in ((64, 32), (128, 16), (128, 16)):
        blocks.append(_pvconv(rng, c, w(cout), R, 2))
        c = w(cout)
    mlps = []
    for cout in (512, 2048):
        mlps.append(_linear(rng, c, w(cout)))
        c = w(cout)
    stages = sum(b.cout for b in blocks) + sum(m.w.shape[0] for m in mlps)
    head, c = [], stages + c
    for cout in (256, 128):
        head.append(_linear(rng, c, w(cout)))
        c = w(cout)
    head.append(_linear(rng, c, 50, final=True))
    return blocks, mlps, head


def _pvcnn2_params(rng, width):
    """The scene PVCNN++: set abstraction and feature propagation levels, head."""
    w = _scale(width)
    sa, skips, c = [], [], 9
    for npoint, radius, pvc, mlp in ((1024, 0.2, (32, 32), (32, 32, 64)),
                                     (256, 0.4, (64, 16), (64, 64, 128)),
                                     (64, 0.8, (128, 8), (128, 128, 256)),
                                     (16, 1.6, None, (256, 256, 512))):
        convs = []
        if pvc:
            convs.append(_pvconv(rng, c, w(pvc[0]), pvc[1], 2))
            c = w(pvc[0])
        skips.append(c)
        layers, ci = [], 3 + c
        for co in mlp:
            layers.append(_linear(rng, ci, w(co)))
            ci = w(co)
        sa.append(SimpleNamespace(pvconvs=convs, npoint=npoint, radius=radius, nsample=32,
                                  mlps=layers))
        c = ci
    fp = []
    for widths, skip in zip(((256, 256), (256, 256), (256, 128), (128, 128, 128)),
                            reversed(skips)):
        layers, ci = [], c + skip
        for co in widths:
            layers.append(_linear(rng, ci, w(co)))
            ci = w(co)
        fp.append(SimpleNamespace(mlps=layers))
        c = ci
    return sa, fp, [_linear(rng, c, w(128)), _linear(rng, w(128), 13, final=True)]


def _head_params(rng, width):
    """The tail alone: the stage widths before it, the MLPs and the head."""
    w = _scale(width)
    stages = [w(64), w(128), w(128)]
    c, mlps = stages[-1], []
    for cout in (512, 2048):
        mlps.append(_linear(rng, c, w(cout)))
        c = w(cout)
    head, c = [], sum(stages) + sum(m.w.shape[0] for m in mlps) + c
    for cout in (256, 128):
        head.append(_linear(rng, c, w(cout)))
        c = w(cout)
    head.append(_linear(rng, c, 50, final=True))
    return stages, mlps, head


def _ceil8(c):
    return -(-c // 8) * 8


def _draw_inputs(case, seed):
    """Everything random of a case, on the host: the same for prepare and exact."""
    rng = np.random.default_rng([int(seed), 977])
    k = case["kind"]
    B, N = case["B"], case["N"]
    d = SimpleNamespace()
    if k in ("layer", "train"):
        bf = case.get("compute", "bf16") == "bf16"
        d.coords = torch.from_numpy(_cloud(rng, case["cloud"], B, N))
        d.feats = _normal(rng, (B, N, case["cin"]))
        if case.get("feat") == "bf16":
            d.feats = d.feats.to(BF16)
        d.layer = _pvconv(rng, case["cin"], case["cout"], case["R"], case.get("convs", 2), bf,
                          case.get("devox", "trilinear"))
        if k == "train":
            d.dout = _normal(rng, (B, N, case["cout"]))
    elif k == "sa":
        d.coords = torch.from_numpy(_cloud(rng, "room", B, N))
        d.feats = _normal(rng, (B, N, case["cin"])).to(BF16)
        d.mlps, c = [], 3 + case["cin"]
        for w in (case["w1"], case["w2"], case["w3"]):
            d.mlps.append(_linear(rng, c, w))
            c = w
    elif k == "fp":
        d.coords = torch.from_numpy(_cloud(rng, "room", B, N))
        d.known = d.coords[:, torch.from_numpy(rng.permutation(N)[:case["M"]])].contiguous()
        d.deep = _normal(rng, (B, case["M"], case["cdeep"])).to(BF16)
        d.skip = _normal(rng, (B, N, case["cskip"])).to(BF16)
        d.mlps, c = [], case["cdeep"] + case["cskip"]
        for _ in range(case["layers"]):
            d.mlps.append(_linear(rng, c, case["width"]))
            c = case["width"]
    elif k == "head":
        d.stages, d.mlps, d.head = _head_params(rng, case["width"])
        d.feats = _normal(rng, (B, N, sum(d.stages))).to(BF16)
    elif k == "pvcnn":
        d.coords = torch.from_numpy(_cloud(rng, "shape", B, N))
        d.feats = d.coords.clone()
        d.blocks, d.mlps, d.head = _pvcnn_params(rng, case["width"])
    else:
        d.coords = torch.from_numpy(_cloud(rng, "room", B, N))
        size = d.coords.amax(1, keepdim=True)
        rgb = torch.from_numpy(rng.random((B, N, 3), dtype=np.float32))
        d.feats = torch.cat([d.coords, rgb, d.coords / size], 2)
        d.sa, d.fp, d.head = _pvcnn2_params(rng, case["width"])
    return d


# --------------------------------------------------------------------------
# what the program holds before the call, and the call
# --------------------------------------------------------------------------
def _dev(t, dtype=None):
    return t.to(DEV) if dtype is None else t.to(dtype).to(DEV)


def _dev_bn(bn):
    return (_dev(bn.gamma), _dev(bn.beta), _dev(bn.mean), _dev(bn.var), bn.eps)


def _dev_linear(lp, pad_to=0):
    w = lp.w
    if pad_to > w.shape[1]:  # zero columns for the rows' padding
        w = torch.cat([w, torch.zeros(w.shape[0], pad_to - w.shape[1])], 1)
    return SimpleNamespace(w=_dev(w, BF16), b=None if lp.b is None else _dev(lp.b),
                           bn=None if lp.bn is None else _dev_bn(lp.bn),
                           act="relu" if lp.relu else "none", cout=w.shape[0])


def prepare(case, seed):
    from paper_1907_03739_amd import binding as pv
    from paper_1907_03739_amd import network as nets
    d = _draw_inputs(case, seed)
    k, B, N = case["kind"], case["B"], case["N"]
    s = dict(kind=k, pv=pv, case=case)
    new = lambda shape, dt: torch.empty(shape, dtype=dt, device=DEV)  # noqa: E731
    if k != "head":
        s["coords"] = _dev(d.coords)
    if k == "layer":
        f32 = case["compute"] == "f32"
        s["feats"] = _dev(d.feats)
        s["layer"] = pv.DeviceLayer(d.layer, DEV, F32 if f32 else BF16)
        s["out"] = new((B, N, case["cout"]), BF16 if case["out"] == "bf16" else F32)
        s["workspace"] = new((max(256, pv.pvconv_forward_workspace_size(B, N, s["layer"])),),
                             torch.uint8)
    elif k == "train":
        L = pv.DeviceLayer(d.layer, DEV, BF16)
        cin, cout, R = case["cin"], case["cout"], case["R"]
        s.update(layer=L, feats=_dev(d.feats), dout=_dev(d.dout),
                 mlp_wt=_dev(d.layer.mlp_w.t().contiguous()))
        V = R ** 3
        s.update(grid=new((B, V, cin), BF16), counts=new((B, V), torch.int32),
                 ids=new((B, N), torch.int32), norm=new((B, N, 3), F32),
                 h1=new((B, V, cout), BF16), h2=new((B, V, cout), BF16),
                 dgrid=new((B, V, cout), F32), dw1=new((cout, 3, 3, 3, cin), F32),
                 dw2=new((cout, 3, 3, 3, cout), F32))
    elif k == "sa":
        M, S, rows = case["M"], case["nsample"], B * case["M"] * case["nsample"]
        wp = _ceil8(3 + case["cin"])
        s.update(feats=_dev(d.feats), idx=new((B, M), torch.int32), centers=new((B, M, 3), F32),
                 ball=new((B, M, S), torch.int32),
                 grouped=torch.zeros((rows, wp), dtype=BF16, device=DEV),
                 mlps=[_dev_linear(m, wp if i == 0 else 0) for i, m in enumerate(d.mlps)],
                 hidden=[new((rows, m.w.shape[0]), BF16) for m in d.mlps],
                 out=new((B * M, case["w3"]), BF16))
    elif k == "fp":
        width = case["cdeep"] + case["cskip"]
        cat = new((B, N, width), BF16)
        cat[:, :, case["cdeep"]:] = _dev(d.skip)
        s.update(known=_dev(d.known), deep=_dev(d.deep), cat=cat,
                 nn_idx=new((B, N, 3), torch.int32), nn_w=new((B, N, 3), F32),
                 mlps=[_dev_linear(m) for m in d.mlps],
                 hidden=[new((B, N, m.w.shape[0]), BF16) for m in d.mlps])
    elif k == "head":
        widths = [m.w.shape[0] for m in d.mlps]
        c0 = sum(d.stages)
        cat = new((B, N, c0 + sum(widths)), BF16)
        cat[:, :, :c0] = _dev(d.feats)
        h0 = d.head[0]
        ns = cat.shape[2]
        s.update(cat=cat, first=(c0 - d.stages[-1], c0), mlps=[_dev_linear(m) for m in d.mlps],
                 slices=[(c0 + sum(widths[:i]), c0 + sum(widths[:i + 1]))
                         for i in range(len(widths))],
                 g=new((B, widths[-1]), F32), row=new((B, h0.w.shape[0]), F32),
                 h0=_dev_linear(SimpleNamespace(w=h0.w[:, :ns].contiguous(), b=None, bn=h0.bn,
                                                relu=True)),
                 h0g=_dev(h0.w[:, ns:].contiguous(), BF16),
                 head=[_dev_linear(m) for m in d.head[1:]],
                 hidden=[new((B, N, m.w.shape[0]), BF16) for m in d.head[:-1]],
                 logits=new((B, N, 50), F32))
    elif k == "pvcnn":
        s["feats"] = _dev(d.feats)
        s["net"] = nets.DeviceNetwork(d.blocks, d.mlps, d.head, B, N, device=DEV)
    else:
        s["feats"] = _dev(d.feats)
        s["net"] = nets.DevicePVCNN2(d.sa, d.fp, d.head, B, N, 9, device=DEV)
    return s


def run(s):
    return _RUN[s["kind"]](s)


def _run_layer(s):
    return s["pv"].pvconv_forward(s["coords"], s["feats"], s["layer"], out=s["out"],
                                  workspace=s["workspace"])


def _run_train(s):
    pv, c, L = s["pv"], s["case"], s["layer"]
    R, w, bn = c["R"], L.conv_w, L.conv_bn
    # forward, keeping what the backward reads
    grid, counts, ids, norm = pv.pvconv_voxelize(
        s["coords"], s["feats"], R, grid_dtype=BF16, grid=s["grid"], counts=s["counts"],
        ids=s["ids"], norm=s["norm"])
    h1 = pv.pvconv_conv3d(grid, w[0], R, bn=bn[0], act="leaky", slope=SLOPE, out=s["h1"])
    h2 = pv.pvconv_conv3d(h1, w[1], R, bn=bn[1], act="leaky", slope=SLOPE, out=s["h2"])
    p = pv.pvconv_point_mlp(s["feats"], L.mlp_w, bn=L.mlp_bn, act="relu")
    y = pv.pvconv_devoxelize(h2, R, norm)
    y += p
    # backward from dL/dy
    dy = s["dout"]
    dg = pv.pvconv_devoxelize_backward(dy, R, norm, out=s["dgrid"])
    dz2 = pv.pvconv_act_bn_backward(dg, h2, bn=bn[1], act="leaky", slope=SLOPE, out=dg).to(BF16)
    dw2 = pv.pvconv_conv3d_backward_weight(dz2, h1, R, out=s["dw2"])
    dh1 = pv.pvconv_conv3d_backward_data(dz2, w[1], R)
    dz1 = pv.pvconv_act_bn_backward(dh1, h1, bn=bn[0], act="leaky", slope=SLOPE,
                                    out=dh1).to(BF16)
    dw1 = pv.pvconv_conv3d_backward_weight(dz1, grid, R, out=s["dw1"])
    dgrid0 = pv.pvconv_conv3d_backward_data(dz1, w[0], R)
    dx = pv.pvconv_voxelize_backward(dgrid0, R, ids, counts)
    dp = pv.pvconv_act_bn_backward(dy, p, bn=L.mlp_bn, act="relu")
    dx += pv.pvconv_point_mlp(dp, s["mlp_wt"], act="none")
    return dict(y=y, dx=dx, dw1=dw1, dw2=dw2)


def _mlps(pv, x, mlps, hidden):
    for m, h in zip(mlps, hidden):
        x = pv.pvconv_point_mlp(x, m.w, bias=m.b, bn=m.bn, act=m.act, out=h)
    return x


def _run_sa(s):
    pv, c = s["pv"], s["case"]
    idx, centers = pv.pvconv_furthest_point_sample(s["coords"], c["M"], idx=s["idx"],
                                                   new_xyz=s["centers"])
    ball = pv.pvconv_ball_query(s["coords"], centers, c["radius"], c["nsample"], idx=s["ball"])
    g = s["grouped"]
    pv.pvconv_group_points(s["coords"], s["feats"], centers, ball, out=g[:, :3 + c["cin"]])
    x = _mlps(pv, g, s["mlps"], s["hidden"])
    return dict(idx=idx, ball=ball, feats=pv.pvconv_group_max(x, c["nsample"], out=s["out"]))


def _run_fp(s):
    pv, c = s["pv"], s["case"]
    idx, w = pv.pvconv_three_nn(s["coords"], s["known"], idx=s["nn_idx"], weight=s["nn_w"])
    pv.pvconv_three_interpolate(s["deep"], idx, w, out=s["cat"][:, :, :c["cdeep"]])
    return dict(idx=idx, weight=w, feats=_mlps(pv, s["cat"], s["mlps"], s["hidden"]))


def _run_head(s):
    pv, cat = s["pv"], s["cat"]
    x = cat[:, :, s["first"][0]:s["first"][1]]
    for m, (a, b) in zip(s["mlps"], s["slices"]):
        x = pv.pvconv_point_mlp(x, m.w, bn=m.bn, act="relu", out=cat[:, :, a:b])
    g = pv.pvconv_maxpool(x, out=s["g"])
    row = pv.pvconv_point_mlp(g, s["h0g"], act="none", out=s["row"])
    m = s["h0"]
    x = pv.pvconv_point_mlp(cat, m.w, bn=m.bn, act="relu", cloud_bias=row,
                            points_per_cloud=cat.shape[1], out=s["hidden"][0])
    return _mlps(pv, x, s["head"], s["hidden"][1:] + [s["logits"]])


def _run_net(s):
    return s["net"].forward(s["coords"], s["feats"])


_RUN = dict(layer=_run_layer, train=_run_train, sa=_run_sa, fp=_run_fp, head=_run_head,
            pvcnn=_run_net, pvcnn2=_run_net)


# --------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct ones may differ
# --------------------------------------------------------------------------
def _layer_work(B, N, cin, cout, R, convs, point_bytes, wsize):
    """Points in and out and the weights; a convolution computes at most every
    voxel, the last one at most the eight corners of every point."""
    V, reach = R ** 3, min(R ** 3, 8 * N)
    flops = 2.0 * B * N * cin * cout
    c, wbytes = cin, cin * cout * wsize
    for i in range(convs):
        flops += 54.0 * B * (reach if i == convs - 1 else V) * c * cout
        wbytes += 27 * c * cout * wsize
        c = cout
    return B * N * (12 + point_bytes) + wbytes, flops


def _mlp_flops(rows, widths):
    return sum(2.0 * rows * a * b for a, b in zip(widths, widths[1:]))


def _mlp_bytes(widths):
    return sum(2.0 * a * b for a, b in zip(widths, widths[1:]))


def _head_widths(width):
    w = _scale(width)
    return [w(64), w(128), w(128)], [w(128), w(512), w(2048)], [w(256), w(128), 50]


def work(case):
    k, B, N = case["kind"], case["B"], case["N"]
    if k == "layer":
        fs = 2 if case["feat"] == "bf16" else 4
        os_ = 2 if case["out"] == "bf16" else 4
        b, f = _layer_work(B, N, case["cin"], case["cout"], case["R"], case["convs"],
                           fs * case["cin"] + os_ * case["cout"],
                           4 if case["compute"] == "f32" else 2)
        return {"bytes": b, "flops": f}
    if k == "train":
        cin, cout, V = case["cin"], case["cout"], case["R"] ** 3
        conv = 54.0 * B * V * cout * (cin + cout)
        # points in, out and their gradients; activations kept once and read
        # once by the backward; weights in, their gradients out
        b = B * N * (12 + 8 * cin + 8 * cout) + B * V * 4.0 * (cin + 2 * cout) + \
            27.0 * cout * (cin + cout) * 6
        return {"bytes": b, "flops": 3 * conv + 6.0 * B * N * cin * cout}
    if k == "sa":
        M, S = case["M"], case["nsample"]
        ws = [3 + case["cin"], case["w1"], case["w2"], case["w3"]]
        b = B * N * (12 + 2 * case["cin"]) + B * M * (4 + 4 * S + 2 * ws[3]) + _mlp_bytes(ws)
        # a distance of every centre to every point, twice (sampling, ball query)
        return {"bytes": b, "flops": _mlp_flops(B * M * S, ws) + 16.0 * B * N * M}
    if k == "fp":
        M = case["M"]
        ws = [case["cdeep"] + case["cskip"]] + [case["width"]] * case["layers"]
        b = B * N * (12 + 24 + 2 * case["cskip"] + 2 * case["width"]) + \
            B * M * (12 + 2 * case["cdeep"]) + _mlp_bytes(ws)
        return {"bytes": b, "flops": _mlp_flops(B * N, ws) + 8.0 * B * N * M}
    st, mw, hw = _head_widths(case["width"])
    hin = sum(st) + sum(mw[1:])
    tail_f = _mlp_flops(B * N, mw) + _mlp_flops(B * N, [hin] + hw) + 2.0 * B * mw[-1] * hw[0]
    tail_b = _mlp_bytes(mw) + _mlp_bytes([hin + mw[-1]] + hw) + B * N * 200.0
    if k == "head":
        return {"bytes": tail_b + B * N * 2.0 * sum(st), "flops": tail_f}
    if k == "pvcnn":
        b, f, c = tail_b, tail_f, 3
        for cout, R in zip(st, (32, 16, 16)):
            lb, lf = _layer_work(B, N, c, cout, R, 2, 0, 2)
            b, f, c = b + lb, f + lf, cout
        return {"bytes": b + B * N * 12.0, "flops": f}
    w = _scale(case["width"])
    n, c, b, f = N, 9, B * N * (36.0 + 52), 0.0
    skip, pts = [], []
    for npoint, pvc, mlp in ((1024, (32, 32), (32, 32, 64)), (256, (64, 16), (64, 64, 128)),
                             (64, (128, 8), (128, 128, 256)), (16, None, (256, 256, 512))):
        if pvc:
            lb, lf = _layer_work(B, n, c, w(pvc[0]), pvc[1], 2, 0, 2)
            b, f, c = b + lb, f + lf, w(pvc[0])
        skip.append(c)
        pts.append(n)
        ws = [3 + c] + [w(m) for m in mlp]
        f += _mlp_flops(B * npoint * 32, ws) + 16.0 * B * n * npoint
        b += _mlp_bytes(ws)
        n, c = npoint, ws[-1]
    for widths, sk, npts in zip(((256, 256), (256, 256), (256, 128), (128, 128, 128)),
                                reversed(skip), reversed(pts)):
        ws = [c + sk] + [w(m) for m in widths]
        f += _mlp_flops(B * npts, ws) + 8.0 * B * npts * n
        b += _mlp_bytes(ws)
        n, c = npts, ws[-1]
    ws = [c, w(128), 13]
    return {"bytes": b + _mlp_bytes(ws), "flops": f + _mlp_flops(B * N, ws)}


def tolerance(case):
    """About four times the measured difference from a 64-bit evaluation: fp32
    sums, bf16 stages between the steps. A training step's gradients differ
    more: an activation within rounding of zero takes either derivative (3 to 4
    per cent measured). Indices are the same integers."""
    k = case["kind"]
    if k == "layer":
        if case["compute"] == "f32":
            return {"rel": 1e-6, "max": 1e-5}
        return {"rel": 6e-3, "max": 0.06}
    if k in ("sa", "fp"):
        return {"rel": 1.1e-2, "max": 0.11, "differ": 0.0}
    if k in ("head", "pvcnn"):
        return {"rel": 1.4e-2, "max": 0.14}
    return {"rel": 3e-2, "max": 0.3 if k == "pvcnn2" else 0.9}


# --------------------------------------------------------------------------
# the same values in 64 bits, from torch alone
# --------------------------------------------------------------------------
def _d(t):
    return t.to(DEV).to(F64)


def _bn64(x, bn):
    if bn is None:
        return x
    return (x - _d(bn.mean)) / torch.sqrt(_d(bn.var) + bn.eps) * _d(bn.gamma) + _d(bn.beta)


def _leaky(x):
    return torch.where(x > 0, x, x * SLOPE)


def _lin64(x, lp):
    y = (x.reshape(-1, x.shape[-1]) @ _d(lp.w).t()).reshape(*x.shape[:-1], -1)
    y = _bn64(y if lp.b is None else y + _d(lp.b), lp.bn)
    return torch.relu(y) if lp.relu else y


def _norm64(coords):
    p = _d(coords)
    p = p - p.mean(1, keepdim=True)
    m = p.square().sum(2).amax(1).sqrt()[:, None, None]
    return torch.where(m > 0, p / (2 * m), torch.zeros_like(p)) + 0.5


def _ids64(pn, R):
    q = torch.floor(pn * R).clamp(0, R - 1).long()
    return (q[..., 0] * R + q[..., 1]) * R + q[..., 2]


def _flat(ids, V):
    return (ids + torch.arange(ids.shape[0], device=ids.device)[:, None] * V).reshape(-1)


def _vox64(feats, ids, R):
    B, N, C = feats.shape
    V = R ** 3
    f = _flat(ids, V)
    n = torch.zeros(B * V, dtype=F64, device=DEV).index_add_(0, f, torch.ones(B * N, dtype=F64,
                                                                              device=DEV))
    g = torch.zeros((B * V, C), dtype=F64, device=DEV).index_add_(0, f, feats.reshape(B * N, C))
    return (g / n.clamp(min=1)[:, None]).view(B, V, C), n


def _windows(x, R):
    """The 27 shifted copies of a zero-padded grid, each [B*V][C]."""
    B, _, C = x.shape
    p = torch.zeros((B, R + 2, R + 2, R + 2, C), dtype=F64, device=DEV)
    p[:, 1:-1, 1:-1, 1:-1] = x.view(B, R, R, R, C)
    for a in range(3):
        for b in range(3):
            for c in range(3):
                yield (a, b, c), p[:, a:a + R, b:b + R, c:c + R].reshape(-1, C)


def _conv64(x, w, R):
    w = _d(w)
    y = torch.zeros((x.shape[0] * R ** 3, w.shape[0]), dtype=F64, device=DEV)
    for (a, b, c), win in _windows(x, R):
        y.addmm_(win, w[:, a, b, c].t())
    return y.view(x.shape[0], -1, w.shape[0])


def _conv64_dw(dy, x, R):
    dw = torch.zeros((dy.shape[2], 3, 3, 3, x.shape[2]), dtype=F64, device=DEV)
    d = dy.reshape(-1, dy.shape[2]).t().contiguous()
    for (a, b, c), win in _windows(x, R):
        dw[:, a, b, c] = d @ win
    return dw


def _corners(pn, R):
    """The eight cells (within the cloud) and weights of every point."""
    t = (pn * R - 0.5).clamp(0, R - 1)
    i0 = t.floor()
    f = t - i0
    i0 = i0.long()
    i1 = (i0 + 1).clamp(max=R - 1)
    for a in (0, 1):
        for b in (0, 1):
            for c in (0, 1):
                u, v, w = ((i1 if s else i0)[..., k] for k, s in enumerate((a, b, c)))
                wt = 1.0
                for k, s in enumerate((a, b, c)):
                    wt = wt * (f[..., k] if s else 1 - f[..., k])
                yield (u * R + v) * R + w, wt


def _devox64(grid, pn, R):
    B, V, C = grid.shape
    g = grid.reshape(B * V, C)
    out = 0
    for cell, wt in _corners(pn, R):
        out = out + g[_flat(cell, V)].view(B, -1, C) * wt[..., None]
    return out


def _pv64(layer, pn, feats):
    """One layer: its output and the states the backward needs."""
    R = layer.R
    ids = _ids64(pn, R)
    h, n = _vox64(feats, ids, R)
    hs = [h]
    for w, bn in zip(layer.conv_w, layer.conv_bn):
        h = _leaky(_bn64(_conv64(h, w, R), bn))
        hs.append(h)
    if layer.devox == "nearest":
        y = h.reshape(-1, h.shape[2])[_flat(ids, R ** 3)].view(*ids.shape, -1)
    else:
        y = _devox64(h, pn, R)
    p = torch.relu(_bn64(feats @ _d(layer.mlp_w).t(), layer.mlp_bn))
    return y + p, hs, ids, n, p


def _train64(layer, pn, feats, dout):
    y, hs, ids, n, p = _pv64(layer, pn, feats)
    R, B = layer.R, feats.shape[0]
    V = R ** 3
    g = torch.zeros((B * V, layer.cout), dtype=F64, device=DEV)
    for cell, wt in _corners(pn, R):
        g.index_add_(0, _flat(cell, V), (dout * wt[..., None]).reshape(-1, layer.cout))
    g = g.view(B, V, layer.cout)
    dws = []
    scale = lambda bn: _d(bn.gamma) / torch.sqrt(_d(bn.var) + bn.eps)  # noqa: E731
    for i in (1, 0):
        g = torch.where(hs[i + 1] > 0, g, g * SLOPE) * scale(layer.conv_bn[i])
        dws.append(_conv64_dw(g, hs[i], R))
        g = _conv64(g, layer.conv_w[i].flip(1, 2, 3).permute(4, 1, 2, 3, 0), R)
    f = _flat(ids, V)
    dx = (g.reshape(B * V, -1)[f] / n[f][:, None]).view(B, -1, layer.cin)
    dp = torch.where(p > 0, dout, torch.zeros_like(dout)) * scale(layer.mlp_bn)
    return dict(y=y, dx=dx + dp @ _d(layer.mlp_w), dw1=dws[1], dw2=dws[0])


def _sq32(a, b):
    """fma(dz, dz, fma(dy, dy, dx*dx)) in float32, the distances that decide an
    index: each product is exact in 64 bits, each sum rounded to 32."""
    d = (a - b)
    x = (d[..., 0] * d[..., 0]).double()
    y, z = d[..., 1].double(), d[..., 2].double()
    return (z * z + (y * y + x).float().double()).float()


def _fps32(xyz, M):
    B, N, _ = xyz.shape
    rows = torch.arange(B, device=DEV)
    best = torch.full((B, N), math.inf, device=DEV)
    at = torch.zeros(B, dtype=torch.long, device=DEV)
    got = [at]
    for _ in range(M - 1):
        best = torch.minimum(best, _sq32(xyz, xyz[rows, at][:, None]))
        at = (best == best.amax(1, keepdim=True)).int().argmax(1)  # ties: the lower index
        got.append(at)
    return torch.stack(got, 1)


def _take(x, idx):
    """x [B][N][C], idx [B][...] -> [B][...][C]."""
    B, N, C = x.shape
    return x.reshape(B * N, C)[_flat(idx.reshape(B, -1), N)].view(*idx.shape, C)


def _ball32(xyz, centers, radius, S):
    r2 = torch.tensor(radius, dtype=F32) * torch.tensor(radius, dtype=F32)
    out = []
    for b in range(xyz.shape[0]):
        inside = _sq32(xyz[b][None], centers[b][:, None]) < r2.to(DEV)
        rank = inside.cumsum(1)
        got = torch.zeros((centers.shape[1], S), dtype=torch.long, device=DEV)
        c, j = torch.nonzero(inside & (rank <= S), as_tuple=True)
        first = torch.where(inside.any(1), inside.int().argmax(1), 0)
        got[:] = first[:, None]
        got[c, rank[c, j] - 1] = j
        out.append(got)
    return torch.stack(out)


def _sa64(xyz, feats, centers, ball, mlps):
    """The features after the maximum, in 64 bits, for given neighbours."""
    x = torch.cat([_d(_take(xyz, ball)) - _d(centers)[:, :, None], _take(feats, ball)], 3)
    for m in mlps:
        x = _lin64(x, m)
    return x.amax(2)


def _nn32(unknown, known):
    """The three nearest known points (ties: the lower index) and their weights."""
    idx = []
    for b in range(unknown.shape[0]):
        d = _sq32(known[b][None], unknown[b][:, None])
        idx.append(torch.sort(d, dim=1, stable=True)[1][:, :3])
    idx = torch.stack(idx)
    dist = (_take(_d(known), idx) - _d(unknown)[:, :, None]).square().sum(3).sqrt()
    w = 1 / (dist + 1e-8)
    return idx, w / w.sum(2, keepdim=True)


def _fp64(xyz, known, deep, skip, mlps):
    idx, w = _nn32(xyz, known)
    x = torch.cat([(_take(deep, idx) * w[..., None]).sum(2), skip], 2)
    for m in mlps:
        x = _lin64(x, m)
    return idx, w, x


def _tail64(stages, last, mlps, head):
    x, every = last, [stages]
    for m in mlps:
        x = _lin64(x, m)
        every.append(x)
    g = x.amax(1, keepdim=True).expand(-1, x.shape[1], -1)
    x = torch.cat(every + [g], 2)
    for m in head:
        x = _lin64(x, m)
    return x


def exact(case, seed):
    d = _draw_inputs(case, seed)
    k = case["kind"]
    feats = _d(d.feats) if k != "fp" else None
    if k == "layer":
        return _pv64(d.layer, _norm64(d.coords), feats)[0]
    if k == "train":
        return _train64(d.layer, _norm64(d.coords), feats, _d(d.dout))
    if k == "head":
        return _tail64(feats, feats[:, :, -d.stages[-1]:], d.mlps, d.head)
    xyz = d.coords.to(DEV)
    if k == "sa":
        idx = _fps32(xyz, case["M"])
        centers = _take(xyz, idx)
        ball = _ball32(xyz, centers, case["radius"], case["nsample"])
        out = _sa64(xyz, feats, centers, ball, d.mlps)
        return dict(idx=idx.int(), ball=ball.int(), feats=out.reshape(-1, case["w3"]))
    if k == "fp":
        idx, w, x = _fp64(xyz, d.known.to(DEV), _d(d.deep), _d(d.skip), d.mlps)
        return dict(idx=idx.int(), weight=w, feats=x)
    if k == "pvcnn":
        pn, x, outs = _norm64(d.coords), feats, []
        for blk in d.blocks:
            x = _pv64(blk, pn, x)[0]
            outs.append(x)
        return _tail64(torch.cat(outs, 2), x, d.mlps, d.head)
    x, pts, skips = feats, [xyz], []
    for lev in d.sa:
        for layer in lev.pvconvs:
            x = _pv64(layer, _norm64(pts[-1]), x)[0]
        skips.append(x)
        centers = _take(pts[-1], _fps32(pts[-1], lev.npoint))
        ball = _ball32(pts[-1], centers, lev.radius, lev.nsample)
        x = _sa64(pts[-1], x, centers, ball, lev.mlps)
        pts.append(centers)
    for lev, l in zip(d.fp, range(len(d.sa) - 1, -1, -1)):
        x = _fp64(pts[l], pts[l + 1], x, skips[l], lev.mlps)[2]
    for m in d.head:
        x = _lin64(x, m)
    return x
