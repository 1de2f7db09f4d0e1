"""Which kernel a GEMM or dK / dV reaches, asked of the library on the host, and the cases of the GPU tests by the kernel they are for.

A form is (kind of tile, how its tiles are walked): kinds by size, "deep" the 128 x 128 tile over a ring of eight slots;
"whole", "split" (every tile's contraction in slices) or "mixed" (whole tiles beside split ones)."""
import paper_2407_20761_amd as ob
import synth_inputs as si

_KINDS = {(256, 256, 4): "big", (192, 256, 4): "mid", (128, 128, 4): "small", (128, 128, 8): "deep", (64, 64, 8): "fine"}


def form(launch):
    how = "whole" if not launch.split_tiles else "mixed" if launch.whole_tiles else "split"
    return _KINDS[launch.tile_rows, launch.tile_cols, launch.ring_slots], how


def forms(layout, M, N, K, scratch=True):
    return [form(p) for p in ob.ob_gemm_plan(layout, M, N, K, scratch)]


def steps(launch, K):
    """K steps of 64 that a workgroup walks: of whole tiles, or of the slices but the last, and of the last"""
    if launch.slices == 1:
        return [(K + 63) // 64]
    return [launch.slice_k // 64, (K - (launch.slices - 1) * launch.slice_k + 63) // 64]


# layout, M, N, K, and the forms they have to have, with scratch
FORMS = [
    (0, 389, 25024, 576, "big whole"), (0, 400, 9344, 4160, "big split"), (0, 646, 22336, 2624, "big mixed"),
    (0, 4608, 4096, 4096, "big mixed"), (0, 1025, 3200, 832, "deep whole"), (0, 300, 2048, 4416, "deep split"),
    (0, 6710, 576, 4928, "deep mixed"), (0, 130, 192, 704, "fine whole"), (0, 200, 768, 4224, "fine split"),
    (0, 2050, 4032, 960, "mid whole"), (0, 4100, 4992, 4096, "mid whole"), (0, 148, 28672, 4096, "mid split"), (0, 5125, 1024, 4160, "mid split"),
    (0, 522, 21952, 4096, "mid mixed"), (0, 1921, 4096, 1088, "small whole"), (0, 65, 16576, 5120, "small split"),
    (0, 7319, 1088, 4096, "small mixed"),
    (1, 389, 25024, 576, "big whole"), (1, 194, 20416, 4096, "big split"), (1, 652, 24576, 2624, "big mixed"),
    (1, 130, 192, 704, "fine whole"), (1, 700, 512, 2112, "fine whole"), (1, 64, 4096, 4224, "fine split"), (1, 1921, 4096, 1088, "mid whole"),
    (1, 526, 4096, 28672, "mid split"), (1, 5125, 1024, 4160, "mid split"), (1, 517, 22720, 4096, "mid mixed"),
    (1, 557, 6144, 576, "small whole"), (1, 33, 8576, 6144, "small split"), (1, 7247, 1088, 5120, "small mixed"),
    (2, 2048, 8128, 900, "big whole"), (2, 704, 6016, 4421, "big split"), (2, 1088, 13312, 3020, "big mixed"),
    (2, 256, 64, 37, "fine whole"), (2, 64, 64, 1000, "fine whole"), (2, 64, 256, 4203, "fine split"), (2, 1664, 640, 1001, "small whole"),
    (2, 768, 512, 3627, "small split"), (2, 24576, 320, 3080, "small mixed"),
    # cut by rows into two launches
    (0, 2049, 8192, 1024, "big whole + fine whole"), (0, 2500, 14336, 1024, "big whole + deep whole"),
    (0, 772, 28672, 1088, "big whole + mid whole"), (0, 1445, 12160, 1024, "mid whole + small whole"),
    (0, 6012, 3072, 2560, "big whole + deep split"), (0, 4211, 4096, 2560, "big whole + fine split"),
    (0, 1442, 12800, 4096, "big whole + mid split"), (0, 4193, 4096, 5120, "big whole + small split"),
    (0, 612, 28672, 12800, "mid whole + big split"),
    (1, 2049, 8192, 1024, "big whole + fine whole"), (1, 2500, 8192, 4160, "big whole + small whole"), (1, 1562, 15168, 1024, "big whole + mid whole"),
    (1, 4911, 3200, 2048, "mid whole + small whole"), (1, 4195, 4096, 2560, "big whole + fine split"),
    (1, 16400, 3200, 3200, "big whole + mid split"), (1, 4494, 4096, 2496, "big whole + small split"),
    (1, 819, 18624, 5760, "mid whole + big split"),
]
# the eight-slot ring of 128 x 128 tiles: "NT", whole and in slices, the numbers of K steps of every remainder modulo the trip's four
DEEP = [(129, 16384, 704), (557, 6144, 768), (557, 5056, 832), (1025, 3200, 832), (300, 8192, 896), (512, 4096, 2496), (512, 4096, 2624), (557, 3072, 2752),
        (300, 2048, 4352), (300, 2048, 4928), (557, 3072, 2816)]
# the hand-over's last GEMM, whose rows are stored through a row list: hidden size on the LLM side, grid, tiles
ROW_LIST = [(64, 4, 16, "fine whole"), (1536, 4, 16, "fine split"), (704, 18, 37, "deep whole"), (2432, 8, 25, "deep split"),
            (384, 32, 22, "small whole"), (2240, 8, 29, "small split"), (1472, 32, 22, "mid whole"), (4096, 32, 5, "mid split"),
            (2112, 32, 22, "big whole"), (2880, 32, 22, "big mixed"), (4096, 32, 17, "big whole + fine whole")]


def named(case_forms):
    return " + ".join(f"{k} {h}" for k, h in case_forms)


def dkv_kernel(lens, nq, nkv, d, mask):
    """the dK / dV kernel of a batch: (key rows of a workgroup, query rows of a streamed tile, threads)"""
    seg = ob.Segments(si.lengths_to_cu(lens), device=None)
    seg.c.cu_dev = 0x1000      # never read: the plan is host work
    plan, _ = ob.ob_varlen_attn_bwd_plan(seg, nq, nkv, d, mask)
    return plan.key_rows, plan.query_rows, ob.ob_varlen_attn_bwd_threads(seg, nq, nkv, d, mask)


# walks of dK / dV: head size, query and key / value heads, segments, and the kernel in which they are walked under each mask
# (bidirectional, causal)
SR64, SR32, SIX = (64, 64, 256), (64, 32, 256), (192, 64, 768)
FOUR, BLOCKS, TWO = (128, 64, 512), (64, 64, 512), (64, 64, 256)
DKV_WALKS = [(64, 2, 1, [4097], SR64, SR64), (64, 2, 1, [8192 + 65], SR64, SR64), (64, 16, 16, [1025] * 3 + [4161], SR32, SR32),
             (64, 10, 10, [4161], SIX, SR64), (128, 2, 1, [4097 + 64], BLOCKS, BLOCKS), (128, 2, 1, [8192 + 65], BLOCKS, BLOCKS),
             (128, 1, 1, [33, 64, 127, 128], TWO, BLOCKS), (128, 3, 1, [65, 129, 193, 321], BLOCKS, BLOCKS), (128, 16, 16, [448], TWO, BLOCKS),
             (128, 32, 8, [4161, 4224] * 2, FOUR, FOUR)]

# activations applied to a GEMM's result on its way out: activation, biases, tokens, hidden, mlp, the tokens more with which they are passes of their own, and
# (tile, ring slots, slices) of the launch, forward and backward
ACTIVATIONS = [(si.MLP_GELU, True, 65, 256, 4160, 2100, ((64, 8, 1), (64, 8, 1))),
               (si.MLP_GELU, True, 1025, 640, 2560, 2200, ((128, 4, 1), (128, 4, 1))),
               (si.MLP_GELU, False, 1500, 768, 2112, 2500, ((128, 8, 1), (128, 4, 1))),
               (si.MLP_SWIGLU, False, 129, 256, 1088, 1700, (None, (64, 8, 1))),
               (si.MLP_SWIGLU, False, 1700, 640, 2560, 1700, (None, (128, 4, 1)))]
