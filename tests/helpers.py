"""Small helpers shared by the tests (no method arithmetic beyond what a pin states itself)."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

from paper_2604_09562_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_09562_amd", "csrc")


def gather_kv(inp, b, kind):
    """Contiguous [kv_len, Hkv, D] float64 view of request b's keys or values.

    Decoding goes through torch's dtype conversions (synth.decode_storage), which
    is independent of the oracle's own C decoders.
    """
    cache = inp["k_cache"] if kind == "k" else inp["v_cache"]
    scale = inp["k_scale"] if kind == "k" else inp["v_scale"]
    L = int(inp["kv_len"][b])
    bs = inp["block_size"]
    nblk = (L + bs - 1) // bs
    ids = inp["block_table"][b, :nblk]
    x = synth.decode_storage(cache[ids], inp["kv_dtype"]).astype(np.float64)  # [nblk,Hkv,bs,D]
    if scale is not None:
        x = x * scale[ids].astype(np.float64)[:, :, None, None]
    x = x.transpose(0, 2, 1, 3).reshape(nblk * bs, inp["num_kv_heads"], inp["head_dim"])
    return x[:L]


def q_values(inp):
    return synth.decode_storage(inp["q"], inp["q_dtype"]).astype(np.float64)


def softmax64(logits, T):
    z = np.asarray(logits, dtype=np.float64) / float(T)
    w = np.exp(z - z.max())
    return w / w.sum()


@functools.lru_cache(maxsize=None)
def _unit_rule_lib():
    """`csrc/unit_rule.h`, compiled for the host."""
    out = tempfile.mkdtemp()
    src, lib = os.path.join(out, "rule.cpp"), os.path.join(out, "rule.so")
    with open(src, "w") as f:
        f.write('#include "unit_rule.h"\n'
                'extern "C" void rule(long long units, int tiles, int rows, int kv8, int cus, int *out)\n'
                '{\n    const ss::AttnUnitChoice c = ss::attn_unit_rule(units, tiles, rows, kv8 != 0, cus);\n'
                '    out[0] = c.splits;\n    out[1] = c.team;\n}\n')
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    fn = ctypes.CDLL(lib).rule
    fn.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_int)]
    return fn


def unit_rule(units, tiles, rows, kv8, cus=256):
    """(workgroups to a unit, wavefronts to a workgroup) of an attention call, (0, 0) if the streaming kernels serve it."""
    out = (ctypes.c_int * 2)()
    _unit_rule_lib()(units, tiles, rows, int(kv8), cus, out)
    return out[0], out[1]


def unit_choice(inp, max_q_len, cus=256):
    """The rule for a matrix-core attention batch of at most 80 query rows a unit whose plan needs no kernel in front, default options."""
    rows = max_q_len * (inp["num_q_heads"] // inp["num_kv_heads"])
    units = inp["batch"] * inp["num_kv_heads"]
    assert rows <= 80
    return (0, 0) if units > 6 * cus else unit_rule(units, inp["max_blocks_per_seq"], rows, inp["kv_dtype"] == "fp8", cus)


def wider(inp, columns):
    """The same batch with a block table of more columns; what stands there may be anything."""
    table = np.full((inp["batch"], columns), 0x7FFFFFFF, np.int32)
    table[:, :inp["block_table"].shape[1]] = inp["block_table"]
    return dict(inp, block_table=table, max_blocks_per_seq=columns)


STREAM_COLUMNS = 1100   # a table that no call of the short-unit kernels has
