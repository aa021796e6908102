"""The library's internal choice of kernel for a call, asked of the host code alone (no GPU: 256 compute units are assumed)."""
import ctypes

from paper_2402_04902_amd import binding


class _LayerDims(ctypes.Structure):  # LayerDims of csrc/l4q_kernels.h
    _fields_ = [("T", ctypes.c_int64), ("i", ctypes.c_int64), ("o", ctypes.c_int64), ("r", ctypes.c_int), ("bits", ctypes.c_int),
                ("g", ctypes.c_int), ("gamma", ctypes.c_float), ("qn", ctypes.c_float), ("qp", ctypes.c_float),
                ("accumulate", ctypes.c_bool)]


class _PrefillPlan(ctypes.Structure):
    _fields_ = [("form", ctypes.c_int), ("us", ctypes.c_double)]


PASSES, TILES_64x128, TILES_128x128, TILES_128x256 = -1, 0, 1, 2


def prompt_plan(T, i, o, bits, g, workspace=True):
    """l4q::qgemm_prompt_plan"""
    f = getattr(binding.load_library(), "_ZN3l4q17qgemm_prompt_planERKNS_9LayerDimsEb")
    f.restype, f.argtypes = _PrefillPlan, [ctypes.POINTER(_LayerDims), ctypes.c_bool]
    q = float(1 << (bits - 1))
    return f(ctypes.byref(_LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False)), workspace)


def prompt_form(*call):
    """The tile shape a quantized forward of more than 64 tokens takes, or PASSES."""
    return prompt_plan(*call).form


def wide_tile_rows(T, i, o, bits, g):
    """l4q::qgemm_prompt_wide_rows: the weight rows of a 128-token wide tile for this call (what TILES_128x256 stands for)."""
    f = getattr(binding.load_library(), "_ZN3l4q22qgemm_prompt_wide_rowsERKNS_9LayerDimsE")
    f.restype, f.argtypes = ctypes.c_int, [ctypes.POINTER(_LayerDims)]
    q = float(1 << (bits - 1))
    return f(ctypes.byref(_LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False)))


class _MergeQuantOut(ctypes.Structure):  # MergeQuantOut<bf16_t> of csrc/l4q_kernels.h
    _fields_ = [("wq", ctypes.c_void_p), ("ld_wq", ctypes.c_int64), ("wqT", ctypes.c_void_p), ("ld_wqT", ctypes.c_int64),
                ("bT", ctypes.c_void_p), ("bT_rank", ctypes.c_int), ("ld_bT", ctypes.c_int64), ("fgrad", ctypes.c_void_p),
                ("codes", ctypes.c_void_p), ("wcomb", ctypes.c_void_p), ("mask", ctypes.c_void_p), ("packed", ctypes.c_void_p),
                ("errors", ctypes.c_void_p), ("init_scale", ctypes.c_void_p), ("init_zero", ctypes.c_void_p),
                ("init_method", ctypes.c_int)]


def merge_quant_transposed(W0, B, scale, zero, bits, g, wqT, bT):
    """l4q::launch_merge_quant<bf16> without a rank term: Wq^T [i, o32] and, where bT [rank, o] is given, B^T."""
    import torch
    f = getattr(binding.load_library(), "_ZN3l4q18launch_merge_quantItEEvRKNS_9LayerDimsEPKT_S6_S6_PKfS8_RKNS_13MergeQuantOutIS4_EEP12ihipStream_t")
    f.restype, f.argtypes = None, [ctypes.c_void_p] * 8
    o, i = W0.shape
    q = float(1 << (bits - 1))
    dims = _LayerDims(1, i, o, 0, bits, g, 1.0, -q, q - 1.0, False)
    out = _MergeQuantOut(wqT=wqT.data_ptr(), ld_wqT=(o + 31) // 32 * 32)
    if bT is not None:
        out.bT, out.bT_rank, out.ld_bT = bT.data_ptr(), B.shape[1], bT.shape[1]
    f(ctypes.byref(dims), W0.data_ptr(), None, B.data_ptr(), scale.data_ptr(), zero.data_ptr(), ctypes.byref(out),
      torch.cuda.current_stream().cuda_stream)


def transposed_rank_product(U, Xs, n_by_r, partial, out):
    """l4q::launch_tn<float, float>: out = U^T Xs [r, n], or its transpose; U [T, r], Xs [T, n], partial ceil(T / 128) r n floats."""
    import torch
    f = getattr(binding.load_library(), "_ZN3l4q9launch_tnIffEEvPKT0_PKT_llibPffS7_bP12ihipStream_t")
    f.restype = None
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_bool, ctypes.c_void_p,
                  ctypes.c_float, ctypes.c_void_p, ctypes.c_bool, ctypes.c_void_p]
    f(U.data_ptr(), Xs.data_ptr(), U.shape[0], Xs.shape[1], U.shape[1], n_by_r, partial.data_ptr(), 1.0, out.data_ptr(), False,
      torch.cuda.current_stream().cuda_stream)


def gpu_us(call, n=30):
    """Time of one call among n, on the GPU."""
    import torch
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(5):
        call()
    t0.record()
    for _ in range(n):
        call()
    t1.record()
    t1.synchronize()
    return 1e3 * t0.elapsed_time(t1) / n


class _BlocksPlan(ctypes.Structure):
    _fields_ = [("nt", ctypes.c_int), ("slices", ctypes.c_int), ("slice_macros", ctypes.c_int), ("us", ctypes.c_double)]


class _WregPlan(ctypes.Structure):
    _fields_ = [("nt", ctypes.c_int), ("cpw", ctypes.c_int), ("grid", ctypes.c_uint), ("wv", ctypes.c_int), ("tbp", ctypes.c_int)]


class _DecodePlan(ctypes.Structure):
    _fields_ = [("nsw", ctypes.c_int), ("xpitch", ctypes.c_int), ("pitch", ctypes.c_int), ("lds", ctypes.c_int)]


class _TilePlan(ctypes.Structure):
    _fields_ = [("tb_max", ctypes.c_int), ("slices", ctypes.c_int), ("klen", ctypes.c_int64), ("pitch", ctypes.c_int * 5),
                ("lds", ctypes.c_int64 * 5)]


class _QgemmRoute(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_int), ("passes", ctypes.c_int), ("blocks", _BlocksPlan * 8), ("prompt", _PrefillPlan),
                ("wreg", _WregPlan), ("decode", _DecodePlan), ("tile", _TilePlan), ("stream_tokens", ctypes.c_int)]


BLOCKS, PROMPT, WREG, DECODE, TILE, STREAM, GENERAL = range(7)  # QgemmKernel


def workspace_bytes(T, i, o, bits, g):
    """What l4q_quantized_forward_workspace_bytes tells."""
    from paper_2402_04902_amd.inputs import DTYPE_BF16, LayerSpec
    return binding.l4q_quantized_forward_workspace_bytes(binding.make_desc(LayerSpec("plan", T, i, o, 8, 16.0, bits, g, DTYPE_BF16)))


def quantized_route(T, i, o, bits, g, workspace):
    """l4q::qgemm_route"""
    f = getattr(binding.load_library(), "_ZN3l4q11qgemm_routeERKNS_9LayerDimsEbPNS_10QgemmRouteE")
    f.restype, f.argtypes = None, [ctypes.POINTER(_LayerDims), ctypes.c_bool, ctypes.POINTER(_QgemmRoute)]
    q, route = float(1 << (bits - 1)), _QgemmRoute()
    f(ctypes.byref(_LayerDims(T, i, o, 8, bits, g, 2.0, -q, q - 1.0, False)), workspace, ctypes.byref(route))
    return route


def quantized_instances(T, i, o, bits, g, workspace):
    """The instances of the quantized forward's kernels (name, template arguments) that a call launches."""
    r = quantized_route(T, i, o, bits, g, workspace)
    if r.kernel == BLOCKS:
        blocks, out = (T + 15) // 16, set()
        for p in range(r.passes):
            t0, t1 = 16 * (blocks * p // r.passes), min(T, 16 * (blocks * (p + 1) // r.passes))
            out.add(("blocks", bits, 64 if bits == 8 or g == 64 else 128, r.blocks[p].nt, (t1 - t0 + 15) // 16))
        return out
    if r.kernel == PROMPT:
        return {("prompt", bits, r.prompt.form)}
    if r.kernel == WREG:
        return {("wreg", bits, r.wreg.nt, r.wreg.cpw, r.wreg.wv)}
    if r.kernel == DECODE:
        return {("decode", bits, r.decode.nsw)}
    if r.kernel == TILE:
        out, step = set(), 16 * r.tile.tb_max
        for t0 in range(0, T, step):
            tb = (min(T - t0, step) + 15) // 16
            while r.tile.lds[tb] == 0:
                tb += 1
            out.add(("tile", bits, tb, r.tile.slices > 1))
        return out
    if r.kernel == STREAM:
        step = r.stream_tokens
        return {("stream", bits, 16 if min(T - t0, step) <= 16 and g % (512 // bits) == 0 else 32) for t0 in range(0, T, step)}
    return {("general", bits, 2 if T > 32 and g >= 64 else 1, g < 64)}
