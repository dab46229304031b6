"""The C-ABI library on the host: loads, exports every declared symbol, agrees
with the oracle on the weight table, and rejects bad arguments before any
launch.  No call here reaches the GPU."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import synth
import paper_2607_26566_amd as t2i
from paper_2607_26566_amd import _lib
from oracle import dit, mmdit

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    names = set()
    for h in os.listdir(os.path.join(ROOT, "include")):
        if not h.endswith(".h"):
            continue
        text = open(os.path.join(ROOT, "include", h)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(t2i_\w+)\s*\(", text))
    return names


def test_library_exports_every_declared_symbol():
    lib = t2i.load()
    declared = declared_functions()
    assert len(declared) >= 16
    for name in declared:
        assert hasattr(lib, name), name
        assert name in _lib.SIGNATURES, name


def test_only_handle_creation_allocates():
    """Steps, samples and cache checks may run where nothing may be allocated:
    the sources name an allocation inside t2i_dit_init alone."""
    src = os.path.join(ROOT, "paper_2607_26566_amd", "csrc")
    found = []
    for f in sorted(os.listdir(src)):
        func = None
        for line in open(os.path.join(src, f)):
            m = re.match(r"[\w:<>*& ]*?\b(\w+)\(", line)   # definitions start in column 0
            if m and line[0].isalpha():
                func = m[1]
            if re.search(r"\bhip\w*Malloc\w*\s*\(", line.split("//")[0]):
                found.append((f, func))
    assert found == [("api.cpp", "t2i_dit_init")]


def test_struct_sizes_match_header_layout():
    # field order and types mirror include/t2i_dit.h; sizes are what the
    # library checks through struct_size
    assert C.sizeof(_lib.t2i_dit_config) == 18 * 4
    assert C.sizeof(_lib.t2i_step_args) % 8 == 0


@pytest.mark.parametrize("name", ["tiny_f32", "dit512", "dit1024_cfg", "packed8"])
def test_weight_table_matches_oracle(name):
    w = synth.workload(name)
    cfg = t2i.Config.from_shape(w)
    assert t2i.weight_table(cfg) == [(n, tuple(s)) for n, s in dit.weight_layout(w)]


def test_mmdit_weight_table_matches_oracle():
    w = synth.workload("mmdit1024")
    cfg = t2i.Config.from_shape(w)
    assert t2i.weight_table(cfg) == [(n, tuple(s)) for n, s in mmdit.weight_layout(w)]


def test_workspace_and_cache_sizes():
    lib = t2i.load()
    w = synth.workload("dit1024_cfg")
    cfg = t2i.Config.from_shape(w)
    ws = lib.t2i_dit_workspace_bytes(cfg.ref())
    # at least the fp32 residual stream and its block-input copy, qkv and fc1 activations
    T, D, F = 8192, 1152, 4608
    assert ws >= T * D * 4 * 2 + T * 3 * D * 2 + T * F * 2
    assert ws < 2 * 1024 ** 3
    toks = (C.c_int32 * 1)(4096)
    cs = lib.t2i_cache_state_bytes(cfg.ref(), 1, toks, 2)
    assert cs >= 4096 * D * 4 * 3
    assert lib.t2i_cache_state_bytes(cfg.ref(), 1, toks, 3) == 0


def test_invalid_configs_are_rejected():
    lib = t2i.load()
    w = synth.workload("dit512")
    for field, bad in [("hidden", 100), ("heads", 7), ("head_dim", 40), ("max_requests", 99),
                       ("dtype", 5), ("patch", 0), ("text_tokens", 0),
                       # bf16 attention operands past 2^31 bytes of addressing
                       ("max_tokens", 1 << 19)]:
        cfg = t2i.Config.from_shape(w)
        setattr(cfg.c, field, bad)
        assert lib.t2i_dit_weight_count(cfg.ref()) == 0, field
        assert lib.t2i_dit_workspace_bytes(cfg.ref()) == 0, field
    cfg = t2i.Config.from_shape(w)
    cfg.c.struct_size = 12
    assert lib.t2i_dit_weight_count(cfg.ref()) == 0


def _fake_handle(w):
    """A handle bound to fake device addresses: valid only for calls that fail
    validation before touching the GPU."""
    lib = t2i.load()
    cfg = t2i.Config.from_shape(w)
    n = lib.t2i_dit_weight_count(cfg.ref())
    ptrs = (C.c_void_p * n)(*[0x1000 * (i + 1) for i in range(n)])
    ws = lib.t2i_dit_workspace_bytes(cfg.ref())
    h = C.c_void_p()
    assert lib.t2i_dit_init(cfg.ref(), ptrs, C.c_void_p(1 << 20), ws - 1, None, C.byref(h)) == 4
    assert lib.t2i_dit_init(cfg.ref(), ptrs, C.c_void_p((1 << 20) + 8), ws, None, C.byref(h)) == 1
    assert lib.t2i_dit_init(cfg.ref(), ptrs, C.c_void_p(1 << 20), ws, None, C.byref(h)) == 0
    return lib, cfg, h


def test_step_argument_errors_return_status():
    w = synth.workload("dit512")
    lib, cfg, h = _fake_handle(w)
    try:
        a = _lib.t2i_step_args()
        a.struct_size = C.sizeof(a) - 8
        assert lib.t2i_dit_step(h, C.byref(a), None) == 1
        a.struct_size = C.sizeof(a)
        a.n_req = 1
        hh = (C.c_int32 * 1)(64)
        ww = (C.c_int32 * 1)(63)                      # not a multiple of the patch
        t = (C.c_double * 1)(1.0)
        a.lat_h, a.lat_w, a.t = hh, ww, t
        a.latents = 0x2000
        a.prompt_embeds = 0x3000
        a.guidance = 1.0
        a.n_blocks = -1
        assert lib.t2i_dit_step(h, C.byref(a), None) == 2
        assert b"multiple of patch" in lib.t2i_last_error(h)
        ww[0] = 64
        a.n_req = 0
        assert lib.t2i_dit_step(h, C.byref(a), None) == 2
        a.n_req = 1
        a.n_blocks = 29
        assert lib.t2i_dit_step(h, C.byref(a), None) == 2
        a.n_blocks = -1
        # callback input: struct size, block order / range, NULL residual
        ctl = _lib.t2i_control()
        ctl.struct_size = C.sizeof(ctl) + 8
        ctl.n = 2
        blocks = (C.c_int32 * 2)(3, 1)
        res = (C.c_void_p * 2)(0x5000, 0x6000)
        ctl.blocks, ctl.residuals, ctl.ready = blocks, res, None
        a.control_outputs = C.cast(C.byref(ctl), C.c_void_p)
        assert lib.t2i_dit_step(h, C.byref(a), None) == 1
        ctl.struct_size = C.sizeof(ctl)
        assert lib.t2i_dit_step(h, C.byref(a), None) == 2          # not increasing
        assert b"increase" in lib.t2i_last_error(h)
        blocks[0], blocks[1] = 1, 28                               # block 28 never runs
        assert lib.t2i_dit_step(h, C.byref(a), None) == 2
        blocks[1] = 3
        res[1] = None
        assert lib.t2i_dit_step(h, C.byref(a), None) == 1
        ctl.n = 0
        assert lib.t2i_dit_step(h, C.byref(a), None) == 2
        a.control_outputs = None
        hh[0] = 128                                     # 4096 tokens > max_tokens 1024
        assert lib.t2i_dit_step(h, C.byref(a), None) == 2
        hh[0] = 64
        t[0] = float("nan")
        assert lib.t2i_dit_step(h, C.byref(a), None) == 1
        a.t = None
        assert lib.t2i_dit_step(h, C.byref(a), None) == 1
    finally:
        lib.t2i_dit_destroy(h)


def test_sample_and_cache_argument_errors():
    w = synth.workload("packed8")
    lib, cfg, h = _fake_handle(w)
    try:
        s = _lib.t2i_sample_args()
        s.struct_size = C.sizeof(s)
        s.n_req = 8
        hs = (C.c_int32 * 8)(*[r[0] for r in w.requests])
        s.lat_h = s.lat_w = hs
        s.latents, s.prompt_embeds = 0x2000, 0x3000
        s.guidance = 1.0
        s.n_steps = 21                                  # > max_steps
        assert lib.t2i_dit_sample(h, C.byref(s), None) == 2
        s.n_steps = 20
        s.start_step = 20
        assert lib.t2i_dit_sample(h, C.byref(s), None) == 2
        s.start_step = 0
        s.cache_tau = 0.1                               # cache without state
        assert lib.t2i_dit_sample(h, C.byref(s), None) == 1
        s.cache_state = 0x5000
        s.cache_state_bytes = 16                        # too small
        assert lib.t2i_dit_sample(h, C.byref(s), None) == 4
        s.cache_mode = 7
        assert lib.t2i_dit_sample(h, C.byref(s), None) == 1
        c = _lib.t2i_cache_args()
        c.struct_size = C.sizeof(c)
        assert lib.t2i_cache_check(h, C.byref(c), None) == 1
    finally:
        lib.t2i_dit_destroy(h)


def test_op_argument_errors():
    lib = t2i.load()
    # bf16 GEMM needs K % 64 == 0
    assert lib.t2i_op_linear(1, 0, 4, 4, 40, 0x1000, 40, 0x2000, 40, 0x3000, 0x4000, 4,
                             None, 0, None, None, None) == 2
    assert b"K % 64" in lib.t2i_ops_last_error()
    assert lib.t2i_op_linear(1, 9, 4, 4, 64, 0x1000, 64, 0x2000, 64, 0x3000, 0x4000, 4,
                             None, 0, None, None, None) == 1
    qs = (C.c_int32 * 1)(0)
    ql = (C.c_int32 * 1)(4)
    kl = (C.c_int32 * 1)(0)                              # no keys
    # LoRA merge: rank range, NULL operand, non-finite alpha
    assert lib.t2i_op_lora_merge(1, 64, 64, 0, 1.0, 0x1000, 64, 0x2000, 0x3000, None) == 2
    assert lib.t2i_op_lora_merge(1, 64, 64, 129, 1.0, 0x1000, 64, 0x2000, 0x3000, None) == 2
    assert lib.t2i_op_lora_merge(1, 64, 64, 8, 1.0, None, 64, 0x2000, 0x3000, None) == 1
    assert lib.t2i_op_lora_merge(1, 64, 64, 8, float("nan"), 0x1000, 64, 0x2000, 0x3000, None) == 1
    assert lib.t2i_op_lora_merge(1, 64, 64, 8, 1.0, 0x1000, 32, 0x2000, 0x3000, None) == 2
    assert lib.t2i_op_attention(1, 2, 72, 1, qs, ql, qs, kl, None, None, 0x1000, 144, 0x2000,
                                144, 0x3000, 144, 0x4000, 144, None) == 2
    assert lib.t2i_op_attention(1, 2, 48, 1, qs, ql, qs, ql, None, None, 0x1000, 96, 0x2000, 96,
                                0x3000, 96, 0x4000, 96, None) == 2
    # no keys in either segment; a second segment given by halves; misaligned segment
    assert lib.t2i_op_attention(1, 2, 72, 1, qs, ql, qs, kl, qs, kl, 0x1000, 144, 0x2000,
                                144, 0x3000, 144, 0x4000, 144, None) == 2
    assert lib.t2i_op_attention(1, 2, 72, 1, qs, ql, qs, ql, qs, None, 0x1000, 144, 0x2000,
                                144, 0x3000, 144, 0x4000, 144, None) == 1
    k2 = (C.c_int32 * 1)(4)
    assert lib.t2i_op_attention(1, 2, 72, 1, qs, ql, qs, ql, k2, ql, 0x1000, 144, 0x2000,
                                144, 0x3000, 144, 0x4000, 144, None) == 2
    # V^T beyond 2^31 bytes of 32-bit offsets (2 heads x 72 rows x ldv x 2 B)
    big = ((1 << 31) // (2 * 2 * 72) + 8) // 8 * 8
    assert lib.t2i_op_attention(1, 2, 72, 1, qs, ql, qs, ql, None, None, 0x1000, 144, 0x2000,
                                144, 0x3000, big, 0x4000, 144, None) == 2
    assert b"2 GiB" in lib.t2i_ops_last_error()
    # cross-attention: bf16 only, at least one key, aligned key start, key range within ldv
    ks8 = (C.c_int32 * 1)(8)
    ks4 = (C.c_int32 * 1)(4)
    assert lib.t2i_op_cross_attention(0, 2, 72, 1, qs, ql, qs, ql, 0x1000, 144, 0x2000, 144,
                                      0x3000, 64, 0x4000, 144, None) == 1
    assert lib.t2i_op_cross_attention(1, 2, 72, 1, qs, ql, qs, kl, 0x1000, 144, 0x2000, 144,
                                      0x3000, 64, 0x4000, 144, None) == 2
    assert lib.t2i_op_cross_attention(1, 2, 72, 1, qs, ql, ks4, ql, 0x1000, 144, 0x2000, 144,
                                      0x3000, 64, 0x4000, 144, None) == 2
    assert lib.t2i_op_cross_attention(1, 2, 72, 1, qs, ql, ks8, ql, 0x1000, 144, 0x2000, 144,
                                      0x3000, 8, 0x4000, 144, None) == 2
    assert lib.t2i_op_cross_attention(1, 2, 48, 1, qs, ql, qs, ql, 0x1000, 96, 0x2000, 96,
                                      0x3000, 64, 0x4000, 96, None) == 2
    assert lib.t2i_op_cross_attention(1, 2, 72, 1, qs, ql, qs, ql, None, 144, 0x2000, 144,
                                      0x3000, 64, 0x4000, 144, None) == 1
    # query projection + cross-attention: the fused setting only where its
    # kernel applies (checked on the host, nothing launched)
    q256 = (C.c_int32 * 1)(256)
    k120 = (C.c_int32 * 1)(120)
    k129 = (C.c_int32 * 1)(129)
    args = lambda fused, hd, qlen, klen, K, qbuf: (
        fused, 16, hd, 1, qs, qlen, qs, klen, K, 0x10000, K, 0x20000, K, 0x30000, 0x40000,
        16 * hd, 0x50000, 128, qbuf, 16 * hd, 0x60000, 16 * hd, None)
    assert lib.t2i_op_linear_cross_attention(*args(2, 72, q256, k120, 1152, None)) == 1
    assert lib.t2i_op_linear_cross_attention(*args(0, 72, q256, k120, 1152, None)) == 1
    assert b"q_buf" in lib.t2i_ops_last_error()
    assert lib.t2i_op_linear_cross_attention(*args(1, 72, q256, k129, 1152, None)) == 2
    assert lib.t2i_op_linear_cross_attention(*args(1, 72, q256, k120, 1000, None)) == 2
    assert lib.t2i_op_linear_cross_attention(*args(1, 72, ql, k120, 1152, None)) == 2
    assert b"fused kernel" in lib.t2i_ops_last_error()
    assert lib.t2i_op_linear_cross_attention(*args(1, 64, q256, k120, 1152, None)) == 2
    assert lib.t2i_op_linear_cross_attention(*args(1, 72, q256, k120, 1088, None)) == 2
    assert b"fused kernel" in lib.t2i_ops_last_error()


@pytest.mark.parametrize("name", ["dit1024_cfg", "mmdit1024", "tiny_f32"])
def test_block_layout_matches_weight_table(name):
    w = synth.workload(name)
    cfg = t2i.Config.from_shape(w)
    first, n, offs, bb = t2i.t2i_dit_block_layout(cfg)
    table = t2i.weight_table(cfg)
    elt = 2 if w.dtype == "bf16" else 4
    assert table[first][0] == "blocks.0.ada.w" or table[first][0] == "blocks.0.txt.ada.w"
    assert table[first + n][0].startswith("blocks.1.")
    end = 0
    for j in range(n):
        size = int(np.prod(table[first + j][1])) * elt
        assert offs[j] % 256 == 0 and offs[j] >= end      # aligned, no overlap
        end = offs[j] + size
        # every block has the same shapes
        assert table[first + (w.depth - 1) * n + j][1] == table[first + j][1]
    assert bb == (end + 255) // 256 * 256
    assert table[first + w.depth * n][0] == "final.ada.w"


def test_residency_argument_errors():
    w = synth.workload("dit512")
    lib, cfg, h = _fake_handle(w)
    try:
        st = (C.c_int32 * w.depth)()
        assert lib.t2i_dit_block_state(h, st) == 0 and list(st) == [0] * w.depth
        # nothing to evict from / load into before a host tier is registered
        assert lib.t2i_dit_evict(h, 3) == 1
        assert b"host tier" in lib.t2i_last_error(h)
        n = C.c_int32(-1)
        assert lib.t2i_dit_load_async(h, None, C.byref(n)) == 1 and n.value == 0
        _, _, _, bb = t2i.t2i_dit_block_layout(cfg)
        need = bb * w.depth
        assert lib.t2i_dit_host_tier(h, None, C.c_void_p(1 << 20), need) == 1
        assert lib.t2i_dit_host_tier(h, C.c_void_p(0x1000), C.c_void_p((1 << 20) + 16), need) == 1
        assert b"aligned" in lib.t2i_last_error(h)
        assert lib.t2i_dit_host_tier(h, C.c_void_p(0x1000), C.c_void_p(1 << 20), need - 1) == 4
        assert lib.t2i_dit_block_state(h, None) == 1
    finally:
        lib.t2i_dit_destroy(h)


def test_static_workspace_init_rejects_configs_beyond_its_size():
    """t2i_dit_init_static checks the config's workspace against the static
    array's size before touching any device: the 1024-px model's is larger."""
    lib = t2i.load()
    w = synth.workload("dit1024_cfg")
    cfg = t2i.Config.from_shape(w)
    need = lib.t2i_dit_workspace_bytes(cfg.ref())
    assert need > (64 << 20)
    n = lib.t2i_dit_weight_count(cfg.ref())
    fake = (C.c_void_p * n)(*([0x1000] * n))
    h = C.c_void_p()
    assert lib.t2i_dit_init_static(cfg.ref(), fake, None, C.byref(h)) == 4   # T2I_ERR_WORKSPACE
    assert not h.value
    assert lib.t2i_dit_init_static(cfg.ref(), fake, None, None) == 1         # out is NULL
    bad = t2i.Config.from_shape(w)
    bad.c.hidden = 100
    assert lib.t2i_dit_init_static(bad.ref(), fake, None, C.byref(h)) == 1


def test_static_workspace_test_configs_fit():
    """The configs the static-workspace GPU test runs stay within the array."""
    lib = t2i.load()
    for name, kw in (("dit1024_cfg", dict(depth=2, requests=((32, 32), (16, 32)))),
                     ("tiny_f32", dict(requests=((16, 16), (16, 8))))):
        cfg = t2i.Config.from_shape(synth.reduced(synth.workload(name), **kw))
        assert 0 < lib.t2i_dit_workspace_bytes(cfg.ref()) <= (64 << 20), name
