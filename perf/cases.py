"""The work that users of the encode library have it do, as measurable cases.

A case is a dict of plain values: which encoder (`model`, one of the repository's own configurations), how many
slices per request (`requests`, "13" or "9,1,6"), through which entry points (`path`) and with which options.

  path "encode"   Encoder.encode: all slices of a batch of requests into one contiguous token buffer
  path "range"    Encoder.encode_range: one encode worker's share [begin, end) of a request
  path "paged"    encode_paged: the tokens go into blocks of a multimodal-token cache
  path "split"    projection on the prefill side: two workers encode halves of a request into their caches
                  (encode_trunk_paged), the prefill side's cache takes the blocks over (transfer_to) and
                  project_merge makes the request's tokens
  path "handover" the encode worker's blocks move to the prefill worker's cache and are read there in token order
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2501_05460_amd import binding as B

BLOCK = 16   # tokens per cache block

# The encoder shapes of the repository's workloads.
_BASE = dict(dtype=1, tile_size=448, patch=14, norm=0, qk_norm=0, act=0, final_norm=0, pixel_shuffle=0, proj_kind=1,
             proj_prenorm=0, eps=1e-6, layer_scale=0, class_token=0, proj_heads=0, mx_fp8=0)
MODELS = {
    "tiny_fp32": dict(_BASE, dtype=0, tile_size=224, hidden=192, heads=3, mlp=768, layers=4, proj_kind=0, proj_mid=0,
                      proj_out=512, max_tiles_per_call=4),
    "siglip": dict(_BASE, hidden=1152, heads=16, mlp=4304, layers=27, act=1, proj_mid=3584, proj_out=3584,
                   max_tiles_per_call=128),
    "siglip_resampler": dict(_BASE, hidden=1152, heads=16, mlp=4304, layers=27, act=1, final_norm=1, proj_kind=2,
                             proj_mid=64, proj_out=3584, proj_heads=28, max_tiles_per_call=128),
    "internvit300m": dict(_BASE, hidden=1024, heads=16, mlp=4096, layers=24, pixel_shuffle=1, proj_prenorm=1,
                          proj_mid=4096, proj_out=4096, max_tiles_per_call=104),
    "internvit300m_cls": dict(_BASE, hidden=1024, heads=16, mlp=4096, layers=24, pixel_shuffle=1, proj_prenorm=1,
                              proj_mid=4096, proj_out=4096, max_tiles_per_call=104, class_token=1, layer_scale=1),
    "internvit6b": dict(_BASE, hidden=3200, heads=25, mlp=12800, layers=45, norm=1, qk_norm=1, pixel_shuffle=1,
                        proj_prenorm=1, proj_mid=5120, proj_out=5120, max_tiles_per_call=40),
}


def listed():
    return [
        # the smallest call: the fp32 configuration, one slice; launches and latency are all of it
        dict(name="tiny_fp32_1", path="encode", model="tiny_fp32", tile=224, requests="1", mx=False),
        # one encode worker's share under intra-request parallelism, one slice of a ten-slice request
        dict(name="siglip_share_1of10", path="range", model="siglip", tile=448, requests="10", begin=4, end=5, mx=False),
        # a quarter of a 13-slice image on the checkpoints' own shape (class token: 1025 tokens, layer scale)
        dict(name="internvit300m_cls_share_3of13", path="range", model="internvit300m_cls", tile=448, requests="13",
             begin=6, end=9, mx=False),
        # a single image request: 12 slices and a thumbnail
        dict(name="internvit300m_13", path="encode", model="internvit300m", tile=448, requests="13", mx=False),
        # the offline batch: eight such images
        dict(name="internvit300m_104", path="encode", model="internvit300m", tile=448, requests="13,13,13,13,13,13,13,13",
             mx=False),
        # a ten-slice request of the SigLIP shape
        dict(name="siglip_10", path="encode", model="siglip", tile=448, requests="10", mx=False),
        # a mixed batch with odd sizes throughout: 378-pixel slices (729 tokens), ragged requests
        dict(name="siglip378_mixed_23", path="encode", model="siglip", tile=378, requests="9,1,6,4,3", mx=False),
        # the resampler projector into a paged cache (64 tokens per slice)
        dict(name="siglip_resampler_paged_10", path="paged", model="siglip_resampler", tile=448, requests="10", mx=False),
        # projection on the prefill side: two workers' halves of a request, merged
        dict(name="internvit300m_split_5", path="split", model="internvit300m", tile=448, requests="5", mx=False),
        # the largest encoder at its full batch
        dict(name="internvit6b_40", path="encode", model="internvit6b", tile=448, requests="40", mx=False),
        # the MXFP8 option on two images
        dict(name="internvit300m_mx_26", path="encode", model="internvit300m", tile=448, requests="13,13", mx=True),
        # hand-over of one image's tokens from the encode worker's cache to the prefill worker's
        dict(name="handover_13", path="handover", model="internvit300m", tile=448, requests="13", mx=False),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def _cut(rng, n):
    """n slices as one to five requests."""
    k = min(n, rng.randint(1, 5))
    cuts = sorted(rng.sample(range(1, n), k - 1)) if k > 1 else []
    edges = [0] + cuts + [n]
    return ",".join(str(b - a) for a, b in zip(edges, edges[1:]))


# Slice sides: 448 mostly, smaller ones where the preprocessor is set to them.  Pixel shuffle needs an even patch
# grid, the block-wise paths a multiple of 16 tokens per slice.
_TILES = {"siglip": [224, 294, 336, 378, 406, 448, 448, 448], "internvit300m": [224, 280, 336, 392, 448, 448, 448],
          "internvit6b": [336, 448, 448]}
_TILES["internvit300m_cls"] = _TILES["internvit300m"]
_TILES_BLOCKS = [224, 336, 392, 448, 448]

# most slices of a drawn call, by encoder: about what the repository's own batches hold, and never more work
# than 40 slices of the largest encoder
_MOST = {"tiny_fp32": 4, "siglip": 64, "siglip_resampler": 32, "internvit300m": 104, "internvit300m_cls": 104,
         "internvit6b": 32}


def draw(rng):
    path = rng.choice(["encode", "encode", "encode", "range", "range", "paged", "split", "handover"])
    if path == "handover":
        return dict(path=path, model=rng.choice(["internvit300m", "siglip", "internvit6b"]), tile=rng.choice([336, 448, 448]),
                    requests=_cut(rng, _log_int(rng, 1, 104)), mx=False)
    if path == "split":
        return dict(path=path, model=rng.choice(["internvit300m", "siglip", "internvit300m_cls"]),
                    tile=rng.choice(_TILES_BLOCKS), requests=str(_log_int(rng, 2, 26)), mx=False)
    if path == "paged":
        model = rng.choice(["siglip_resampler", "siglip", "internvit300m"])
        tile = 448 if model == "siglip_resampler" else rng.choice([448, 448, 224])
        return dict(path=path, model=model, tile=tile, requests=_cut(rng, _log_int(rng, 1, 32)), mx=False)
    model = rng.choice(["tiny_fp32", "siglip", "siglip", "siglip_resampler", "internvit300m", "internvit300m_cls",
                        "internvit6b"])
    n = _log_int(rng, 1, _MOST[model])
    tile = rng.choice(_TILES.get(model, [MODELS[model]["tile_size"]]))
    mx = model not in ("tiny_fp32", "siglip_resampler") and rng.random() < 0.2
    if path == "range":
        begin = rng.randint(0, 5)
        return dict(path=path, model=model, tile=tile, requests=str(begin + n + rng.randint(0, 5)), begin=begin,
                    end=begin + n, mx=mx)
    return dict(path=path, model=model, tile=tile, requests=_cut(rng, n), mx=mx)


def _desc(case):
    return SimpleNamespace(**dict(MODELS[case["model"]], tile_size=case["tile"], mx_fp8=int(bool(case["mx"]))))


def _counts(case):
    return [int(v) for v in case["requests"].split(",")]


def _dims(d):
    patches = (d.tile_size // d.patch) ** 2
    n_out = d.proj_mid if d.proj_kind == 2 else patches // 4 if d.pixel_shuffle else patches
    return patches, n_out, d.hidden * (4 if d.pixel_shuffle else 1)


def _weight_specs(d):
    """(shape, kind) of every tensor in the order the library takes them; kind: w matrix / bias / embedding,
    g norm gain, b norm shift, s layer scale."""
    D, F = d.hidden, d.mlp
    patches, _, pin = _dims(d)
    s = [((D, 3 * d.patch * d.patch), "w"), ((D,), "w"), ((patches + d.class_token, D), "w")]
    norm = [((D,), "g")] + ([((D,), "b")] if d.norm == 0 else [])
    if d.class_token:
        s.append(((D,), "w"))
    for _ in range(d.layers):
        s += norm + [((3 * D, D), "w"), ((3 * D,), "w")]
        if d.qk_norm:
            s += [((D if d.qk_norm == 1 else D // d.heads,), "g")] * 2
        s += [((D, D), "w"), ((D,), "w")] + ([((D,), "s")] if d.layer_scale else [])
        s += norm + [((F, D), "w"), ((F,), "w"), ((D, F), "w"), ((D,), "w")] + ([((D,), "s")] if d.layer_scale else [])
    if d.final_norm:
        s += norm
    if d.proj_prenorm:
        s += [((pin,), "g"), ((pin,), "b")]
    if d.proj_kind == 2:
        E, Q = d.proj_out, d.proj_mid
        ln = [((E,), "g"), ((E,), "b")]
        s += [((E, D), "w"), ((Q, E), "w"), ((patches, E), "w")] + ln + ln
        s += [((3 * E, E), "w"), ((3 * E,), "w"), ((E, E), "w"), ((E,), "w")] + ln + [((E, E), "w")]
    elif d.proj_kind == 0:
        s += [((d.proj_out, pin), "w"), ((d.proj_out,), "w")]
    else:
        s += [((d.proj_mid, pin), "w"), ((d.proj_mid,), "w"), ((d.proj_out, d.proj_mid), "w"), ((d.proj_out,), "w")]
    return s


def _weights(d, gen):
    dtype = torch.bfloat16 if d.dtype == 1 else torch.float32
    out = []
    for shape, kind in _weight_specs(d):
        if kind == "s":
            t = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(0.9).add_(0.1)
        else:
            t = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(0.02)
            if kind == "g":
                t.add_(1.0)
        out.append(t.to(dtype))
    return out


def _cache_of(d, n_blocks, width):
    return B.MMCache(n_blocks, BLOCK, width, d.dtype == 1)


def prepare(case, seed):
    """The worker's encoder (weights packed once), the request's slices as the preprocessor leaves them, the token
    buffer or caches with their pre-allocated blocks."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    d, counts = _desc(case), _counts(case)
    n = sum(counts)
    patches, n_out, _ = _dims(d)
    st = SimpleNamespace(path=case["path"], n=n, offsets=[0] + list(np.cumsum(counts).tolist()))
    if st.path == "handover":
        blocks = n * n_out // BLOCK
        spare = blocks // 4 + 8   # the caches also hold other requests' tokens: the ids are scattered
        st.src, st.dst = (_cache_of(d, blocks + spare, d.proj_out) for _ in range(2))
        order = np.random.default_rng(seed)
        st.src_ids, st.dst_ids = [], []
        for cache, ids in ((st.src, st.src_ids), (st.dst, st.dst_ids)):
            taken = cache.alloc((blocks + spare) * BLOCK)
            ids.extend(int(v) for v in order.permutation(taken)[:blocks])
        pool = st.src.pool_tensor()
        pool.copy_(torch.randn(pool.shape, generator=gen, device="cuda", dtype=pool.dtype))
        return st
    st.enc = B.Encoder(d, _weights(d, gen))
    st.tiles = torch.rand((n, 3, d.tile_size, d.tile_size), generator=gen, device="cuda").mul_(2.0).sub_(1.0)
    if st.path == "range":
        st.begin, st.end = case["begin"], case["end"]
    if st.path == "paged":
        per = n_out // BLOCK
        st.cache = _cache_of(d, n * per, d.proj_out)
        st.tables = [st.cache.alloc(k * n_out) for k in counts]
        st.cache.pool_tensor().zero_()
    elif st.path == "split":
        per = patches // BLOCK
        st.half = n // 2
        st.workers = [_cache_of(d, k * per, d.hidden) for k in (st.half, n - st.half)]
        st.worker_ids = [w.alloc(k * patches) for w, k in zip(st.workers, (st.half, n - st.half))]
        st.prefill = _cache_of(d, n * per, d.hidden)
        st.prefill_ids = st.prefill.alloc(n * patches)
        st.cut = st.half * per
        st.out = st.enc.alloc_out(n)
    else:
        st.out = st.enc.alloc_out(n)
    return st


def run(st):
    if st.path == "encode":
        return st.enc.encode(st.tiles, st.offsets, st.out)
    if st.path == "range":
        st.enc.encode_range(st.tiles, st.begin, st.end, st.out)
        per = st.enc.tokens_per_tile
        return st.out[st.begin * per:st.end * per]
    if st.path == "paged":
        B.encode_paged(st.enc, st.tiles, st.offsets, st.cache, st.tables)
        pool = st.cache.pool_tensor()
        pool.cache = st.cache   # a view of the cache's memory: whoever holds the output holds the cache
        return pool
    if st.path == "split":
        B.encode_trunk_paged(st.enc, st.tiles, 0, st.half, st.workers[0], st.worker_ids[0])
        B.encode_trunk_paged(st.enc, st.tiles, st.half, st.n, st.workers[1], st.worker_ids[1])
        st.workers[0].transfer_to(st.worker_ids[0], st.prefill, st.prefill_ids[:st.cut])
        st.workers[1].transfer_to(st.worker_ids[1], st.prefill, st.prefill_ids[st.cut:])
        return B.project_merge(st.enc, st.prefill, st.prefill_ids, st.n, st.out)
    st.src.transfer_to(st.src_ids, st.dst, st.dst_ids)
    return st.dst.gather(st.dst_ids)


def work(case):
    d, counts = _desc(case), _counts(case)
    n = sum(counts)
    patches, n_out, pin = _dims(d)
    size = 2 if d.dtype == 1 else 4
    if case["path"] == "handover":
        return {"bytes": 3 * n * n_out * d.proj_out * size, "flops": 0}   # source read, pool and reader's buffer written
    if case["path"] == "range":
        n = case["end"] - case["begin"]
    D, F, L, tok = d.hidden, d.mlp, d.layers, patches + d.class_token
    flops = 2 * patches * 3 * d.patch * d.patch * D + L * (8 * tok * D * D + 4 * tok * D * F + 4 * tok * tok * D)
    if d.proj_kind == 2:
        E = d.proj_out
        flops += 2 * patches * D * E + 4 * patches * E * E + 4 * n_out * patches * E + 4 * n_out * E * E
    elif d.proj_kind == 0:
        flops += 2 * n_out * pin * d.proj_out
    else:
        flops += 2 * n_out * pin * d.proj_mid + 2 * n_out * d.proj_mid * d.proj_out
    weights = sum(math.prod(shape) for shape, _ in _weight_specs(d)) * size
    moved = weights + n * (3 * d.tile_size * d.tile_size * 4 + n_out * d.proj_out * size)
    if case["path"] == "split":
        moved += 4 * n * patches * D * size   # workers' caches written and read, prefill cache written and read
    return {"bytes": moved, "flops": n * flops}


def tolerance(case):
    """Relative L2 error another correct implementation would show.  Measured: pixels moved by one part in 2^22, which
    re-draws every rounding behind them, change the fp32 encoder's output by 5.4e-7, the bf16 encoders' by 3.3e-3 (the
    resampler) to 6.5e-3 (against 5.0e-3 to 6.0e-3 between bf16 and fp32 mode on the same weights) and the MXFP8
    option's by 7.3e-2 to 8.0e-2: an element next to a rounding boundary takes the neighbouring value, and the depth of
    the encoders makes two independent draws of the rounding noise of it."""
    if case["path"] == "handover":
        return "exact"
    if MODELS[case["model"]]["dtype"] == 0:
        return {"rel": 4e-6}
    return {"rel": 2.4e-1} if case["mx"] else {"rel": 2e-2}


def _exact_norm(x, w, kind, eps):
    if kind == 0:
        g, b = next(w), next(w)
        return torch.nn.functional.layer_norm(x, (x.shape[-1],), g, b, eps)
    return x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + eps) * next(w)


def _exact_gelu(x, tanh=False):
    return torch.nn.functional.gelu(x, approximate="tanh" if tanh else "none")


def _exact_attention(q, k, v, heads):
    """q [Q, E], k and v [N, E] of one slice."""
    hd = q.shape[-1] // heads
    q, k, v = (t.reshape(t.shape[0], heads, hd).transpose(0, 1).contiguous() for t in (q, k, v))
    p = torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(hd), dim=-1)
    return torch.matmul(p, v).transpose(0, 1).reshape(-1, heads * hd)


def exact(case, seed):
    """The tokens of `run` by the textbook definitions in float64.  The MXFP8 option has none: its result is that of
    rounded codes, and two computations of it decorrelate over the layers."""
    if case["path"] == "handover" or case["mx"]:
        return None
    d, F = _desc(case), torch.nn.functional
    gen = torch.Generator(device="cuda").manual_seed(seed)
    raw = _weights(d, gen)
    n = sum(_counts(case))
    tiles = torch.rand((n, 3, d.tile_size, d.tile_size), generator=gen, device="cuda").mul_(2.0).sub_(1.0)
    if case["path"] == "range":
        tiles = tiles[case["begin"]:case["end"]]
        n = len(tiles)
    patches, n_out, pin = _dims(d)
    D, g, P = d.hidden, d.tile_size // d.patch, d.patch
    w = (t.double() for t in raw)   # in the order of _weight_specs, one at a time
    a = tiles.double().reshape(n, 3, g, P, g, P).permute(0, 2, 4, 1, 3, 5).reshape(n * patches, 3 * P * P)
    x = F.linear(a, next(w), next(w)).reshape(n, patches, D)
    pos = next(w)
    if d.class_token:
        x = torch.cat([next(w).expand(n, 1, D), x], dim=1)
    x = x + pos
    del a, tiles
    for _ in range(d.layers):
        u = _exact_norm(x, w, d.norm, d.eps)
        q, k, v = F.linear(u, next(w), next(w)).split(D, dim=-1)
        if d.qk_norm:   # 1: over all heads together, 2: by head
            hd = D if d.qk_norm == 1 else D // d.heads
            q, k = (_exact_norm(t.reshape(-1, hd), w, 1, d.eps).reshape(t.shape) for t in (q, k))
        o = torch.stack([_exact_attention(q[t], k[t], v[t], d.heads) for t in range(n)])
        o = F.linear(o, next(w), next(w))
        x = x + (o * next(w) if d.layer_scale else o)
        del u, q, k, v, o
        u = F.linear(_exact_norm(x, w, d.norm, d.eps), next(w), next(w))
        u = F.linear(_exact_gelu(u, d.act == 1), next(w), next(w))
        x = x + (u * next(w) if d.layer_scale else u)
        del u
    if d.final_norm:
        x = _exact_norm(x, w, d.norm, d.eps)
    x = x[:, d.class_token:]
    if d.pixel_shuffle:
        x = x.reshape(n, g // 2, 2, g // 2, 2, D).permute(0, 1, 3, 2, 4, 5).reshape(n, n_out, pin)
    if d.proj_prenorm:
        x = _exact_norm(x, w, 0, d.eps)
    if d.proj_kind == 2:
        E = d.proj_out
        kv, query, r_pos = F.linear(x, next(w)), next(w), next(w)
        query, kv = (_exact_norm(t, w, 0, d.eps) for t in (query, kv))
        in_w, in_b = next(w).split(E), next(w).split(E)
        query = F.linear(query, in_w[0], in_b[0])
        k, v = F.linear(kv + r_pos, in_w[1], in_b[1]), F.linear(kv, in_w[2], in_b[2])
        x = torch.stack([_exact_attention(query, k[t], v[t], d.proj_heads) for t in range(n)])
        x = F.linear(_exact_norm(F.linear(x, next(w), next(w)), w, 0, d.eps), next(w))
    elif d.proj_kind == 0:
        x = F.linear(x, next(w), next(w))
    else:
        x = F.linear(_exact_gelu(F.linear(x, next(w), next(w))), next(w), next(w))
    return x.reshape(-1, BLOCK, d.proj_out) if case["path"] == "paged" else x.reshape(-1, d.proj_out)
