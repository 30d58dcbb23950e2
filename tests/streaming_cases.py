"""Steps whose w and m are streamed: one large layer and ragged ones (a layer
of 7, 63, 1 and of 2049 elements, so that groups end after 1, 3 and 7
elements), every flag combination.  (MiB of w and m, K, dtype, options)."""
from paper_2603_18112_amd import layouts

SD = layouts.LAYER_SCALE | layouts.LAYER_DECAY

STEP = [
    (9, 16, "f32", dict(small_replica=-1)),
    (9, 17, "f32", dict(small_replica=16)),
    (9, 32, "bf16", dict()),
    (9, 33, "bf16", dict(small_replica=-1)),
    (9, 64, "bf16", dict(small_replica=63)),
    (130, 8, "f32", dict(small_replica=7)),
    (130, 9, "f32", dict(mode="static", static_scale=1.7)),
    (258, 1, "f32", dict()),
    (258, 2, "f32", dict(small_replica=1)),
    (258, 3, "f32", dict(small_replica=-1)),
    (514, 4, "f32", dict(mode="sgd")),
]
ELEMENT_SCALES = [
    (130, 16, "f32", dict(small_replica=-1)),
    (130, 17, "f32", dict(small_replica=16)),
]
LARS = [
    (66, 5, "f32", dict(reuse_w_norms=True)),
    (66, 8, "f32", dict(small_replica=7)),
    (66, 7, "bf16", dict(reuse_w_norms=True, small_replica=-1)),
    (66, 16, "bf16", dict()),
    (514, 3, "f32", dict(reuse_w_norms=True)),
]


def layout(mib):
    sizes = [mib * (1 << 17) - 4096, 7, 2049, 63, 1703, 1]
    flags = [SD, layouts.LAYER_SCALE, 0, layouts.LAYER_DECAY, SD, SD]
    return layouts.custom_layout(sizes, flags, pad=8)


def name(case):
    mib, K, dtype, hyper = case
    return f"{mib}MiB-K{K}-{dtype}-" + "-".join(f"{k}={v}" for k, v in hyper.items())
