"""Host-side checks of the C ABI: the library loads, exports every declared
symbol, and refuses bad arguments before anything is launched (no GPU needed)."""
import ctypes
import os
import re

import pytest

import paper_2101_03961_amd as sw
from paper_2101_03961_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "switchffn.h")


def _declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(switch_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = ctypes.CDLL(sw.library_path())
    names = _declared_functions()
    assert {"switch_forward", "switch_backward", "switch_capacity", "switch_workspace_size",
            "switch_status_string"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_capacity_and_workspace_host_functions():
    cases = {(256, 4, 1.25): 80, (65536, 128, 1.0): 512, (65536, 128, 1.25): 640,
             (16384, 64, 1.25): 320, (32768, 64, 1.0): 512, (10, 3, 1.0): 3, (5, 8, 1.0): 0}
    for (T, E, cf), C in cases.items():
        cfg = sw.SwitchConfig(T, 64, 256, E, cf, 0.01, sw.SW_F32)
        assert sw.switch_capacity(cfg) == C
        assert sw.switch_workspace_size(cfg) > 0
    # routing groups: Eq. 3 on the group's tokens; one group when the field is 0 or 1
    for n, C in {0: 512, 1: 512, 8: 64, 128: 4, 512: 1, 1024: 0}.items():
        cfg = sw.SwitchConfig(65536, 64, 256, 128, 1.0, 0.01, sw.SW_BF16, 0, n)
        assert sw.switch_capacity(cfg) == C
        assert sw.switch_workspace_size(cfg) > 0
    a = sw.switch_workspace_size(sw.SwitchConfig(4096, 64, 256, 8, 1.0, 0.01, sw.SW_BF16))
    b = sw.switch_workspace_size(sw.SwitchConfig(4096, 64, 256, 8, 2.0, 0.01, sw.SW_BF16))
    assert b > a


@pytest.mark.parametrize("kw,status", [
    (dict(T=-1), -2), (dict(T=2**31), -2), (dict(E=0), -2), (dict(E=5000), -2), (dict(d_model=0), -2),
    (dict(d_model=12), -2),            # bf16 rows must be whole 16-byte chunks
    (dict(d_ff=100), -2),
    (dict(capacity_factor=0.0), -3), (dict(capacity_factor=-1.0), -3),
    (dict(capacity_factor=float("nan")), -3), (dict(capacity_factor=float("inf")), -3),
    (dict(alpha=float("nan")), -3), (dict(act_dtype=7), -4),
    (dict(n_groups=3), -2),            # 256 tokens do not split into 3 groups
    (dict(d_model=65536, d_ff=32768), -2),   # one expert's bf16 matrix would reach 4 GB
    (dict(n_groups=-1), -2),
    (dict(ffn_kind=2), -4), (dict(ffn_kind=-1), -4),
    (dict(ffn_kind=1, d_model=32768, d_ff=16384), -2),   # [W_g | W_l] of one expert reaches 2 GB
    (dict(ntlb_rounds=-1), -3), (dict(ntlb_rounds=17), -3),
    (dict(expert_dropout=1.0), -3), (dict(expert_dropout=-0.1), -3),
    (dict(expert_dropout=float("nan")), -3),
    (dict(jitter_eps=1.0), -3), (dict(jitter_eps=-1e-3), -3), (dict(jitter_eps=float("nan")), -3),
    (dict(flags=2), -3), (dict(flags=-1), -3),   # only the documented flag bits
])
def test_bad_config_is_refused(kw, status):
    assert ctypes.sizeof(sw.SwitchConfig) == 88       # the header's struct
    base = dict(T=256, d_model=64, d_ff=256, E=4, capacity_factor=1.25, alpha=0.01,
                act_dtype=sw.SW_BF16, ffn_kind=0, n_groups=1, expert_dropout=0.0, jitter_eps=0.0,
                seed=0, ntlb_rounds=0, flags=0)
    base.update(kw)
    cfg = sw.SwitchConfig(*[base[k] for k in ("T", "d_model", "d_ff", "E", "capacity_factor",
                                              "alpha", "act_dtype", "ffn_kind", "n_groups",
                                              "expert_dropout", "jitter_eps", "seed", "ntlb_rounds",
                                              "flags")])
    with pytest.raises(sw.SwitchError) as ei:
        sw.switch_capacity(cfg)
    assert ei.value.status == status
    with pytest.raises(sw.SwitchError):
        sw.switch_workspace_size(cfg)
    # forward / backward refuse the same configuration before looking at pointers
    assert sw.switch_forward(cfg, *([None] * 13), None, 0, check=False) == status
    assert sw.switch_backward(cfg, None, 1.0, *([None] * 10), None, 0, check=False) == status
    assert sw.switch_forward_static(cfg, *([None] * 13), check=False) == status


def test_null_misaligned_and_small_workspace_are_refused():
    cfg = sw.SwitchConfig(256, 64, 256, 4, 1.25, 0.01, sw.SW_F32)
    need = sw.switch_workspace_size(cfg)
    ok = 0x1000  # fake, aligned, never dereferenced: checks run before any launch
    args = [ok] * 13
    assert sw.switch_forward(cfg, *([None] + args[1:]), ok, need, check=False) == -1   # x NULL
    assert sw.switch_forward(cfg, *([ok + 4] + args[1:]), ok, need, check=False) == -6  # misaligned
    args_nl = list(args)
    args_nl[12] = None                                                                  # logits optional
    assert sw.switch_forward(cfg, *args_nl, None, need, check=False) == -5              # no workspace
    assert sw.switch_forward(cfg, *args_nl, ok, need - 1, check=False) == -5            # too small
    assert sw.switch_forward(cfg, *args_nl, ok + 16, need, check=False) == -5           # misaligned ws
    bargs = [ok] * 10
    assert sw.switch_backward(cfg, None, 1.0, *bargs, ok, need, check=False) == -1
    assert sw.switch_backward(cfg, ok, float("nan"), *bargs, ok, need, check=False) == -3
    assert sw.switch_backward(cfg, ok, 1.0, *bargs, ok, 16, check=False) == -5


def test_vector_read_pointers_must_be_aligned():
    """b_r is read 16 bytes at a time by the matrix-core router beyond 128 experts, db_r is
    written by whole chunks: both are covered by the alignment check."""
    cfg = sw.SwitchConfig(256, 64, 256, 4, 1.25, 0.01, sw.SW_F32)
    need = sw.switch_workspace_size(cfg)
    ok = 0x1000
    args = [ok] * 13
    args[2] = ok + 4                                                                    # b_r
    assert sw.switch_forward(cfg, *args, ok, need, check=False) == -6
    assert sw.switch_forward_static(cfg, *args, check=False) == -6
    bargs = [ok] * 10
    bargs[7] = ok + 8                                                                   # db_r
    assert sw.switch_backward(cfg, ok, 1.0, *bargs, ok, need, check=False) == -6


def test_static_scratch_variant_refuses_what_does_not_fit():
    """The size limit depends on the configuration alone and is checked first; NULL and
    misaligned pointers are refused like in switch_forward; all before any launch."""
    big = sw.SwitchConfig(65536, 768, 3072, 128, 1.0, 0.01, sw.SW_BF16)
    assert sw.switch_workspace_size(big) > sw.SW_STATIC_SCRATCH_BYTES
    assert sw.switch_forward_static(big, *([None] * 13), check=False) == -9
    text = open(HEADER).read()
    m = re.search(r"#define SW_STATIC_SCRATCH_BYTES \((\d+)u \* 1024u \* 1024u\)", text)
    assert m and int(m.group(1)) * 1024 * 1024 == sw.SW_STATIC_SCRATCH_BYTES
    small = sw.SwitchConfig(256, 64, 256, 4, 1.25, 0.01, sw.SW_F32)
    assert sw.switch_workspace_size(small) <= sw.SW_STATIC_SCRATCH_BYTES
    ok = 0x1000
    assert sw.switch_forward_static(small, *([None] + [ok] * 12), check=False) == -1
    assert sw.switch_forward_static(small, *([ok + 4] + [ok] * 12), check=False) == -6
    assert "static scratch" in sw.switch_status_string(-9)


def _workspace_with_square_tiles(T, d, f, E, C_g, n, bf16, geglu, jitter, ntlb):
    """Bytes of the workspace as it was laid out when every bf16 GEMM ran on 256 x 256 tiles and nothing
    shared memory: what decided which layers switch_forward_static takes."""
    up = lambda v, a: -(-v // a) * a
    tiles = lambda v, a: -(-v // a)
    f1, C, nb, elt = (2 * f if geglu else f), n * C_g, n * tiles(T // n, 256), 2 if bf16 else 4
    dpad, et = up(d, 32), tiles(E, 128)
    jit = bf16 and jitter
    dpad_r = 3 * dpad if jit else dpad
    splits = tiles(T, up(tiles(T, 85), 64) or 64)
    parts = [T * E * 4, T * 4, T * 4, nb * 256 * 4] + 3 * [nb * E * 4] + [E * 4] + 3 * [n * E * 4] + [64, E * 4]
    parts += [(E * C + 128) * 4, E * C * 4, (E * C + 128) * 4, T * 4, E * C * d * elt]
    parts += [E * C * f1 * elt if geglu else 0, E * C * f * elt, E * C * d * elt, E * C * d * elt]
    parts += [E * C * f * elt if geglu else 0, E * C * f1 * elt, E * C * d * elt]
    parts += [T * 4, T * E * 4, min(nb, 64) * d * E * 4, tiles(T, 256) * E * 4]
    parts += [et * 3 * 128 * dpad_r * 2, et * d * 512, et * T * 512, T * dpad_r * 2 if jit else 0, T * 4 if jit else 0]
    parts += [et * splits * (2 * dpad if jit else d) * 1024, E * tiles(f, 256) * tiles(C, 256) * 8192]
    if ntlb:
        parts += [T * E * 4, T * 4] + 4 * [n * E * 4]
    return sum(up(p, 256) for p in parts)


# The static scratch takes every layer that it took with 256 x 256 tiles alone: other tiles may pad the ReLU
# bits further and the router's token blocks are smaller, but no workspace of that size has grown.
def test_static_scratch_variant_keeps_what_fits():
    import random
    rng = random.Random(20)
    lu = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    # (T, d, f, E, cf, jitter, ntlb, n): bits padded by a tall or wide tile, many experts, capacity 0
    near = [(335, 200, 9712, 57, 1.0, 0.01, 0, 1), (236, 168, 7792, 64, 2.0, 0.01, 0, 1), (209, 264, 2704, 263, 2.0, 0, 0, 1),
            (503, 264, 2000, 308, 1.0, 0, 0, 1), (412, 264, 1960, 317, 1.25, 0, 0, 1), (87, 216, 2744, 284, 4.0, 0, 0, 1),
            (85, 272, 2472, 316, 4.0, 0, 0, 1), (174, 272, 1984, 330, 2.0, 0, 1, 1), (57, 16, 17264, 2, 7.8947369, 0, 0, 1),
            (29, 16, 31096, 1, 8.827586215, 0, 0, 1), (64, 32, 31512, 1, 4.000000004, 0, 0, 64),
            (7898, 8, 60000, 216, 2.7e-4, 0, 1, 1)]
    cases = [(T, d, f, E, cf, 1, 0, j, r, n) for T, d, f, E, cf, j, r, n in near]
    while len(cases) < 30000:
        n = rng.choice((1, 1, 1, 2, 7, 64, 500))
        T = n * rng.choice((lu(1, 40000 // n), 1, 64, 65, 66, 193))
        d, E, C = 8 * lu(1, 64), lu(1, 512), rng.choice((0, 0, 1, 2, lu(1, 300), 225, 256))   # C slots per expert and group
        dtype, geglu, jitter, ntlb = rng.choice((1, 1, 1, 0)), rng.choice((0, 0, 0, 1)), rng.choice((0.0, 0.0, 0.01)), rng.choice((0, 0, 1))
        if T > 60000 or E * C * n * (4 * d + 16) * 2 > sw.SW_STATIC_SCRATCH_BYTES:
            continue
        # d_ff that brings the whole close to the limit
        at8, at8008 = (_workspace_with_square_tiles(T, d, f, E, C, n, dtype, geglu, jitter > 0, ntlb) for f in (8, 8008))
        f = int((sw.SW_STATIC_SCRATCH_BYTES * rng.uniform(0.9, 1.0) - at8) * 8000 / max(at8008 - at8, 1))
        cases.append((T, d, min(max(8, f // 8 * 8), 60000), E, max(C, 0.01) * E * n / T * (1 + 1e-9), dtype, geglu, jitter, ntlb, n))
    fitted = 0
    for T, d, f, E, cf, dtype, geglu, jitter, ntlb, n in cases:
        cfg = sw.SwitchConfig(T, d, f, E, cf, 0.01, dtype, geglu, n, 0.0, jitter, 1, ntlb, 0)
        size = sw.switch_workspace_size(cfg)
        before = _workspace_with_square_tiles(T, d, f, E, sw.switch_capacity(cfg), n, dtype, geglu, jitter > 0, ntlb)
        if before <= sw.SW_STATIC_SCRATCH_BYTES:
            fitted += 1
            assert size <= before, (T, d, f, E, cf, dtype, geglu, jitter, ntlb, n, before, size)
    assert fitted > 10000


@pytest.mark.parametrize("T,d,f,E,cf,dtype,jitter", [
    (262, 2584, 10248, 6, 2.0, "bf16", 0.0), (1050, 512, 1856, 16, 2.0, "bf16", 0.0), (1050, 512, 2304, 16, 2.0, "bf16", 0.0),
    (1024, 512, 2048, 16, 2.0, "bf16", 0.01), (700, 768, 3072, 16, 1.25, "bf16", 0.01), (1050, 512, 1024, 16, 2.0, "f32", 0.0),
    (65536, 768, 3072, 128, 1.0, "bf16", 0.0), (256, 64, 256, 4, 1.25, "f32", 0.0)])
def test_workspace_size_is_what_the_passes_ask_for(T, d, f, E, cf, dtype, jitter):
    """Not a byte more: one less is refused, by both passes, and the static scratch takes a layer if and only if it fits."""
    cfg = sw.SwitchConfig(T, d, f, E, cf, 0.01, sw.SW_BF16 if dtype == "bf16" else sw.SW_F32, 0, 1, 0.0, jitter)
    need, ok = sw.switch_workspace_size(cfg), 0x1000   # (pointers are not followed: the checks come first)
    assert sw.switch_forward(cfg, *([ok] * 13), ok, need - 1, check=False) == -5
    assert sw.switch_backward(cfg, ok, 1.0, *([ok] * 10), ok, need - 1, check=False) == -5
    fits = need <= sw.SW_STATIC_SCRATCH_BYTES
    assert sw.switch_forward_static(cfg, None, *([ok] * 12), check=False) == (-1 if fits else -9)


def test_status_strings():
    assert sw.switch_status_string(0) == "ok"
    seen = {sw.switch_status_string(s) for s in range(-9, 1)}
    assert len(seen) == 10
    assert "unknown" in sw.switch_status_string(-99)


def test_binding_has_no_fallback_path():
    """The Python side only marshals arguments: it must not import the oracle
    or implement the layer itself."""
    for mod in ("binding.py", "layer.py", "__init__.py"):
        src = open(os.path.join(os.path.dirname(binding.__file__), mod)).read()
        assert "import oracle" not in src and "from oracle" not in src
        assert "softmax" not in src and "matmul" not in src and "einsum" not in src
