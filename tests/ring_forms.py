"""Which tile form of the many-row kernel a launch takes, from the cost table in gemm.hip, and decoders
whose launches reach every form at its column remainders (no tests here)."""
from __future__ import annotations

import os
import re
from dataclasses import replace

import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_22641_amd", "csrc")


def forms():
    """(mi, nj, kb, ns, fit, us) of RING_FORMS: tiles of 32 mi rows x 32 nj columns, K steps of 32 kb."""
    with open(os.path.join(CSRC, "gemm.hip")) as f:
        table = re.search(r"RING_FORMS\[\w+\] = \{(.*?)\n\};", f.read(), re.S).group(1)
    rows = re.findall(r"\{(\d+), (\d+), (\d+), (\d+), (\d+), \{([^}]*)\}\}", table)
    return [tuple(int(v) for v in r[:5]) + ([float(v) for v in r[5].split(",")],) for r in rows]


def ring_shape(width, M, K, can_split, cus=256):
    """(form, K ranges): ring_shape of gemm.hip."""
    best, best_t = (0, 1), None
    for f, (mi, nj, kb, _, fit, us) in enumerate(forms()):
        tiles = -(-M // (32 * mi)) * -(-width // (32 * nj))
        for S in range(1, (4 if can_split else 1) + 1):
            nk = K // 32 // kb
            per = -(-nk // S)
            if per * (S - 1) >= nk:
                break
            full, rest = divmod(-(-tiles * S // cus), fit)
            t = per * kb * (full * us[fit - 1] + (us[rest - 1] if rest else 0.0))
            if S > 1:
                t += 3.0 + M * width * (S + 4) * 4.0 / 6.0e6
            if best_t is None or t < best_t:
                best, best_t = (f, S), t
    return best


def _wl(name, arch, batch, gamma, d_model, n_heads, d_ff, vocab, **kw):
    base, wl = (synth.SMALL_T5_BF16, synth.S_T5) if arch == "t5" else (synth.SMALL_LLAMA_BF16, synth.S_LLAMA)
    sh = replace(base, name=name, n_layers=2, d_model=d_model, n_heads=n_heads, d_head=64, d_ff=d_ff, vocab=vocab, **kw)
    return wl.with_(name=name, shape=sh, batch=batch, prompt_len=3, draft_layers=1, gamma=gamma,
                    new_tokens=2 * gamma + 4, deep_scale=1.0)


# Few inputs and many outputs (or the reverse), so that the oracle is quick.  Widths end one 64-column
# block (a vocabulary, 7 or more columns) past the wider tiles, rows inside a tile.
WORKLOADS = [
    _wl("rows-600-wide", "llama", 24, 24, 64, 103, 10304, 20601, n_visual=4),
    _wl("rows-129-wide", "t5", 43, 2, 64, 43, 12352, 24711, n_visual=8),
    _wl("rows-129-k1088", "llama", 43, 2, 1856, 17, 1088, 999, n_visual=4),
    _wl("rows-260-k2112", "llama", 52, 4, 4416, 3, 2112, 1500, n_visual=4),
    _wl("rows-900-k4160", "llama", 36, 24, 3136, 3, 4160, 1500, n_visual=4),
    _wl("rows-130-imitation", "t5", 130, 1, 64, 87, 320, 8327, n_visual=8, in_hidden=24768),
]


def launches(wl):
    """(kind, M, width, tiled columns, K, can split) of a verify pass's, a draft's and a T5 prefill's
    many-row launches."""
    sh, M = wl.shape, wl.batch * (wl.gamma + 1)
    D, HD, F = sh.d_model, sh.hd, sh.d_ff
    out = [("qkv", M, 3 * HD, 3 * HD, D, False), ("resid", M, D, D, HD, True), ("gated", M, 2 * F, 2 * F, D, False),
           ("resid", M, D, D, F, True), ("argmax", M, sh.vocab, sh.vocab, D, False)]
    if sh.arch == "t5":
        MV, n_tab = wl.batch * sh.n_visual, 2 * sh.n_layers
        out += [("store", M, HD, HD, D, False), ("cross", MV, HD * n_tab, HD, D, False)]
    if wl.batch > 128:
        out += [("bias-gelu", wl.batch, sh.in_width, sh.in_width, D, False),
                ("bias-resid", wl.batch, D, D, sh.in_width, False)]
    return [l for l in out if l[1] > 128]


def covered(cus=256):
    """(kind, form's tile width, column remainder, 'whole' / 'split' / 'uneven') of all launches."""
    seen = set()
    for wl in WORKLOADS:
        for kind, M, width, cols, K, split in launches(wl):
            f, S = ring_shape(width, M, K, split, cus)
            mi, nj, kb = forms()[f][:3]
            nk = K // 32 // kb
            ranges = "whole" if S == 1 else ("split" if nk % S == 0 else "uneven")
            seen.add((wl.name, kind, f, cols % (32 * nj) != 0, ranges))
    return seen


def stress_last_columns(w):
    """Weights that read the last 64 columns of each wide projection, times 8 (exact in bfloat16)."""
    for n in ("lm_head", "in_w2"):
        w[n][:, -64:] *= 8
    for lw in w["layers"]:
        for n in ("wo", "xo", "w_down"):
            if n in lw and lw[n].shape[1] > 64:
                lw[n][:, -64:] *= 8
