"""The split-operand kernels: layers that the compute calls run on them
instead of on a tile plan (conv_fwd_split_plan).

CPU: the kernels' index maps emulated from the exported launch fields (every
staged slot an operand reads is written, every output stored once, the sum
equal to the oracle), for every staging mode, strides, padding, tails of
channels, rows and columns.  GPU: every compiled instance, on a layer that is
routed to it, against the oracle and (fp32) against the tile plan, whose error
in the 2-norm it must not exceed; bf16 Out, infinities and NaNs, extreme
magnitudes, unaligned tensors, graph capture and tuning.
"""
import os
import re

import numpy as np
import pytest
import torch

from oracle import conv as oconv
from paper_2101_09808_amd import conv as B
from paper_2101_09808_amd.workloads import ConvShape, make_inputs

DEV = "cuda:0"
CONV, IMAGE, POINT = 0, 1, 2


def split_plan(s):
    return B.conv_fwd_split_plan(*s.key(), s.stride, s.pad, B.CONV_DTYPE_BF16 if s.dtype == "bf16" else B.CONV_DTYPE_F32)


def oracle(s, In, Ker):
    return oconv.conv_fwd_ex(In.float().numpy(), Ker.float().numpy(), (s.stride,) * 2, (s.pad,) * 2)


# ----------------------------------------------------------------- CPU

def units(s, g, m):
    """(octet of the chunk, tap) of the four lane groups of MFMA step m;
    image mode: (kernel row, first of two columns)."""
    for u in range(4 * m, 4 * m + 4):
        if g["mode"] == IMAGE:
            sp = (s.S + 1) // 2
            yield u // sp, 2 * (u % sp)
        else:
            yield u % g["co"], u // g["co"]


def stage_vec(s, g, In, lds, ch, nu0, q0):
    """Items of four neighbouring input pixels; columns in the padding zeroed."""
    N, C, K, H, W, R, S = s.key()
    st, pd = s.stride, s.pad
    x0 = q0 * st - pd
    xa = max(x0, 0) & (~0 if g["npl"] == 3 else ~1)
    ph = st if g["nb"] > 1 else 1
    for o in range(g["co"]):
        for e in range(g["E"]):
            f, x = e // g["in_wp"] // g["in_rows"], e % g["in_wp"]
            if not 0 <= x0 + x * st + f % g["nb"] < W:
                lds[o * g["Epad"] + e] = 0
    E4 = g["na"] * g["in_rows"] * g["ng"]
    for it in range(g["items"]):
        o, e = it // E4, it % E4
        pr, gi = e // g["ng"], e % g["ng"]
        a, row = pr // g["in_rows"], pr % g["in_rows"]
        n, yi = divmod(nu0 + row, g["Hi"])
        y, base = yi * st + a - pd, min(xa + 4 * gi, W - 4)
        assert 0 <= base and base + 4 <= W and (g["npl"] == 3 or (((n * C * H + y) * W + base) % 2 == 0))
        c0 = (ch * g["co"] + o) * 8
        m = max(0, min(8, C - c0))
        for p in range(4):
            v = base + p - x0
            b, ix = v % ph, v // ph
            if v < 0 or ix >= g["in_wp"]:
                continue
            vec = np.zeros(8)
            if n < N and 0 <= y < H:
                vec[:m] = In[n, c0:c0 + m, y, base + p]
            lds[o * g["Epad"] + ((a * g["nb"] + b) * g["in_rows"] + row) * g["in_wp"] + ix] = vec


def emulate(s, g, In, Ker, wgs):
    """Out and store counts of the given workgroups, in float64."""
    N, C, K, H, W, R, S = s.key()
    P, Q = s.P, s.Q
    st, pd = s.stride, s.pad
    out, written = np.zeros((N, K, P, Q)), np.zeros((N, K, P, Q), int)
    point, image = g["mode"] == POINT, g["mode"] == IMAGE
    BK, BP = 16 * g["wk"] * g["nwk"], 16 * g["wp"] * g["nwp"]
    Cp = g["nchunks"] * g["co"] * 8
    for b in wgs:
        G8 = g["num_tiles"] & ~7
        L = (b & 7) * (G8 >> 3) + (b >> 3) if b < G8 else b
        if g["order"] == 0:
            kt, rest = L % g["tiles_k"], L // g["tiles_k"]
            ct, rt = rest % g["tiles_cols"], rest // g["tiles_cols"]
        else:
            ct, rest = L % g["tiles_cols"], L // g["tiles_cols"]
            rt, kt = rest % g["tiles_rows"], rest // g["tiles_rows"]
        rho0, rho_end = rt * g["tr"], min((rt + 1) * g["tr"], N * P)
        q0 = ct * g["tw"]
        n0 = rho0 // P
        nu0 = n0 * g["Hi"] + (rho0 - n0 * P) * g["rm"]
        # packed rows: Ker rows, or pixels of In
        prow = np.arange(BK) + (rt if point else kt) * BK
        acc = np.zeros((BK, BP))
        for ch in range(g["nchunks"]):
            lds = np.full(((g["co"] + 1) * g["Epad"], 8), np.nan)
            zeros = g["npl"] == 1 and 4 * g["steps"] > g["co"] * R * S  # an octet for the units past the last tap
            if zeros:
                lds[g["co"] * g["Epad"]:] = 0
                assert g["buf_bytes"] == 16 * len(lds)
            if g["vec"] > 1:
                stage_vec(s, g, In, lds, ch, nu0, q0)
            for it in range(g["items"] if g["vec"] == 1 else 0):
                v = np.zeros(8)
                if point:
                    e, o = it // g["co"], it % g["co"]
                    k = kt * BP + e
                    c0 = (ch * g["co"] + o) * 8
                    if k < K:
                        n = max(0, min(8, C - c0))
                        v[:n] = Ker[k, c0:c0 + n, 0, 0]
                else:
                    o, e = it // g["E"], it % g["E"]
                    pr, x = e // g["in_wp"], e % g["in_wp"]
                    f, row = pr // g["in_rows"], pr % g["in_rows"]
                    a, bb = f // g["nb"], f % g["nb"]
                    n, yi = divmod(nu0 + row, g["Hi"])
                    if image:
                        for p in range(2):
                            y, xx = yi - pd, q0 * st + 2 * x + p - pd
                            if n < N and 0 <= y < H and 0 <= xx < W:
                                v[4 * p:4 * p + C] = In[n, :, y, xx]
                    else:
                        y, xx = yi * st + a - pd, (q0 + x) * st + bb - pd
                        c0 = (ch * g["co"] + o) * 8
                        if n < N and 0 <= y < H and 0 <= xx < W:
                            m = max(0, min(8, C - c0))
                            v[:m] = In[n, c0:c0 + m, y, xx]
                lds[o * g["Epad"] + e] = v
            assert g["items"] <= g["ni"] * 64 * g["nwk"] * g["nwp"] * g["nwc"]
            flat = lds.reshape(-1)
            for m in range(g["steps"]):
                for uu in units(s, g, m):
                    A = np.zeros((BK, 8))
                    if image:
                        r, s0 = uu
                        off = 2 * 4 * (r * g["in_wp"] + s0 // 2) if r < R else 0
                        for i, k in enumerate(prow):
                            if k < K and r < R:
                                for e in range(8):
                                    if e % 4 < C and s0 + e // 4 < S:
                                        A[i, e] = Ker[k, e % 4, r, s0 + e // 4]
                    else:
                        o, tap = uu
                        real = o < g["co"] and tap < (1 if point else R * S)
                        t = tap if real and not point else 0
                        r, ss = t // S, t % S
                        off = 8 * (o * g["Epad"] + ((r % st * g["nb"] + ss % st) * g["in_rows"] + r // st) * g["in_wp"]
                                   + ss // st)
                        if zeros and not real:
                            off = 8 * g["co"] * g["Epad"]
                        c0 = (ch * g["co"] + o) * 8
                        for i, k in enumerate(prow):
                            n = max(0, min(8, C - c0))
                            if not real:
                                continue
                            if point and k < N * P * Q:
                                A[i, :n] = In[k // (P * Q), c0:c0 + n].reshape(n, -1)[:, k % (P * Q)]
                            elif not point and k < K:
                                A[i, :n] = Ker[k, c0:c0 + n, r, ss]
                    for p in range(BP):
                        if point:
                            ad = 8 * p
                        else:
                            t, col = divmod(p, g["tw"])
                            rho = rho0 + t
                            if t >= g["tr"] or rho >= rho_end:
                                continue
                            n, h = divmod(rho, P)
                            row = n * g["Hi"] + h * g["rm"] - nu0
                            ad = 8 * row * g["in_wp"] + (4 * col * g["cm"] if image else 8 * col)
                        vec = flat[ad + off:ad + off + 8]
                        q = q0 + (p % g["tw"])
                        if (p < BP and point) or q < Q:
                            assert not np.isnan(vec).any(), "reads a slot that no item writes"
                            acc[:, p] += A @ vec
        for p in range(BP):
            if point:
                k = kt * BP + p
                for i, px in enumerate(prow):
                    if k < K and px < N * P * Q:
                        n, x = divmod(px, P * Q)
                        out[n, k, x // Q, x % Q] = acc[i, p]
                        written[n, k, x // Q, x % Q] += 1
                continue
            t, col = divmod(p, g["tw"])
            rho, q = rho0 + t, q0 + col
            if t >= g["tr"] or rho >= rho_end or q >= Q:
                continue
            n, h = divmod(rho, P)
            for i, k in enumerate(prow):
                if k < K:
                    out[n, k, h, q] = acc[i, p]
                    written[n, k, h, q] += 1
    return out, written


# Layers on the route, for each staging mode: strides 1 and 2, padding, tails
# of channels, output channels, rows and columns, tiles across images.
EMULATED = [
    ConvShape("sp_bf16_3x3_tails", 2, 20, 24, 9, 11, 3, 3, "bf16", 701, 1, 1),
    ConvShape("sp_bf16_3x3_s2", 2, 12, 20, 13, 10, 3, 3, "bf16", 702, 2, 1),
    ConvShape("sp_bf16_1x1", 2, 40, 24, 7, 9, 1, 1, "bf16", 703),
    ConvShape("sp_bf16_1x1_s2", 3, 17, 20, 9, 9, 1, 1, "bf16", 704, 2, 0),
    ConvShape("sp_bf16_3x3_c64", 1, 64, 40, 8, 10, 3, 3, "bf16", 705),
    # four pixels per load: K <= 32 and more, padded, a tail of columns
    ConvShape("sp_bf16_vec_k32", 9, 32, 32, 60, 50, 3, 3, "bf16", 706),
    ConvShape("sp_bf16_vec_k32_pad", 5, 30, 24, 70, 62, 3, 3, "bf16", 707, 1, 1),
    # units past the last tap: 18 of 20, 50 of 52, 35 of 36
    ConvShape("sp_bf16_s2_c3", 1, 3, 7, 56, 61, 3, 3, "bf16", 708, 2, 0),
    ConvShape("sp_bf16_5x5_c17", 1, 17, 7, 7, 6, 5, 5, "bf16", 709),
    ConvShape("sp_bf16_7x5", 8, 8, 200, 43, 63, 7, 5, "bf16", 710, 3, 1),
]


@pytest.mark.parametrize("s", EMULATED, ids=lambda s: s.name)
def test_index_maps(s):
    g = split_plan(s)
    assert g and g["lds_bytes"] <= 160 * 1024
    In, Ker = make_inputs(s)
    T = g["num_tiles"]
    some = range(T) if T <= 16 else sorted({0, 1, T // 3, T // 2, T - 2, T - 1})
    out, written = emulate(s, g, In.double().numpy(), Ker.double().numpy(), some)
    hit = written == 1
    assert written.max() == 1 and (hit.all() if T <= 16 else hit.any())
    ref = oracle(s, In, Ker)
    assert np.max(np.abs((out - ref)[hit])) <= 1e-9 * np.max(np.abs(ref))


# larger layers, first, middle and last workgroups
SAMPLED = [
    ConvShape("sp_f32_3x3_c128", 32, 128, 128, 30, 30, 3, 3, "f32", 711),
    ConvShape("sp_f32_3x3_c512", 32, 512, 512, 9, 9, 3, 3, "f32", 712),
    ConvShape("sp_f32_3x3s2p1", 32, 64, 128, 56, 56, 3, 3, "f32", 713, 2, 1),
    ConvShape("sp_f32_image_7x7s2", 32, 3, 64, 224, 224, 7, 7, "f32", 714, 2, 3),
    ConvShape("sp_f32_image_3x3s2", 32, 3, 64, 224, 224, 3, 3, "f32", 715, 2, 1),
    ConvShape("sp_f32_point", 1, 1024, 28269, 17, 17, 1, 1, "f32", 716),
    ConvShape("sp_f32_1x1_c464", 2, 464, 176, 60, 60, 1, 1, "f32", 717),
    ConvShape("sp_f32_3x3_odd", 23, 181, 92, 19, 19, 3, 3, "f32", 718),
]


@pytest.mark.parametrize("s", SAMPLED, ids=lambda s: s.name)
def test_sampled_workgroups(s):
    g = split_plan(s)
    assert g
    In, Ker = make_inputs(s)
    T = g["num_tiles"]
    few = dict(g, nchunks=1) if g["nchunks"] > 1 else g  # the first chunk of channels: the others only move the channel
    nc = few["nchunks"] * g["co"] * 8 if g["mode"] != IMAGE else s.C
    s1 = ConvShape(s.name, s.N, min(nc, s.C), s.K, s.H, s.W, s.R, s.S, s.dtype, s.seed, s.stride, s.pad)
    In1, Ker1 = In[:, :nc].contiguous(), Ker[:, :nc].contiguous()
    out, written = emulate(s1, few, In1.double().numpy(), Ker1.double().numpy(), sorted({0, T // 2, T - 1}))
    hit = written == 1
    assert written.max() == 1 and hit.any()
    n = sorted(set(np.nonzero(hit)[0]))
    sn = ConvShape(s.name, len(n), s1.C, s.K, s.H, s.W, s.R, s.S, s.dtype, s.seed, s.stride, s.pad)
    ref = oracle(sn, In1[n].contiguous(), Ker1)
    assert np.max(np.abs((out[n] - ref)[hit[n]])) <= 1e-9 * np.max(np.abs(ref))


def test_route_needs_a_plan():
    """A layer without a plan stays refused (7x7 taps, stride 1, three channels)."""
    dims = (5, 3, 32, 220, 220, 7, 7)
    with pytest.raises(B.ConvError) as e:
        B.conv_fwd_ex_plan(*dims, 1, 3)
    assert e.value.status == B.CONV_ENOPLAN
    assert B.conv_fwd_split_plan(*dims, 1, 3) is None


def test_a_missing_plan_is_remembered():
    """bf16 layers without a bf16 plan (5x5 taps) look that up on every call:
    it must not search the plans again each time (17 us)."""
    import ctypes
    import time

    L, plan = B.lib(), B.ConvPlan()

    def best(dims, status):
        t = []
        for _ in range(200):
            a = time.perf_counter()
            st = L.conv_fwd_plan(*dims, B.CONV_DTYPE_BF16, ctypes.byref(plan))
            t.append(time.perf_counter() - a)
            assert st == status
        return min(t)
    assert best((2, 24, 40, 14, 12, 5, 5), B.CONV_ENOPLAN) <= 4 * best((2, 24, 40, 14, 12, 3, 3), B.CONV_OK)


@pytest.mark.parametrize("s", [
    # fp32 layers with taps of less than about 27 us
    ConvShape("", 2, 112, 464, 31, 31, 3, 3, "f32", 0), ConvShape("", 5, 64, 32, 11, 15, 3, 3, "f32", 0, 2, 1),
    ConvShape("", 2, 23, 96, 11, 11, 3, 3, "f32", 0, 1, 1), ConvShape("", 4, 17, 32, 26, 26, 3, 3, "f32", 0),
    ConvShape("", 6, 3, 32, 147, 147, 3, 3, "f32", 0, 1, 1), ConvShape("", 9, 64, 176, 11, 11, 3, 3, "f32", 0, 2, 1),
    ConvShape("", 1, 160, 21, 27, 27, 3, 3, "f32", 0, 2, 1), ConvShape("", 6, 64, 853, 10, 10, 3, 3, "f32", 0, 1, 1),
    # bf16 layers of one chunk below 13.2 us
    ConvShape("", 2, 27, 391, 8, 8, 3, 3, "bf16", 0), ConvShape("", 3, 16, 447, 16, 16, 3, 3, "bf16", 0),
], ids=str)
def test_layers_that_are_faster_on_their_plans(s):
    """Random layers that ran at 0.87 to 0.96 of their plans' speed on the
    split kernels stay on their plans."""
    assert split_plan(s) is None


@pytest.mark.parametrize("dims", [(298261, 1, 2, 60, 60, 5, 5), (65535, 1, 2, 128, 128, 5, 5),
                                  (1369568, 1, 2, 28, 28, 5, 5)], ids=str)
def test_grid_fits_a_launch(dims):
    """A grid dimension takes fewer than 2^32 threads: layers whose split grid
    would be larger stay on the widened fp32 plan."""
    g = B.conv_fwd_split_plan(*dims, dtype=B.CONV_DTYPE_BF16)
    assert g is None or g["num_tiles"] * 64 * g["nwk"] * g["nwp"] * g["nwc"] < 2 ** 32
    plan = B.conv_fwd_plan(*dims)  # of the widened inputs
    assert plan["num_wg"] * B.conv_fwd_geometry(*dims, plan)["threads"] < 2 ** 32


# ----------------------------------------------------------------- GPU

def say(*a):
    print(*a, flush=True)


def run(s, In, Ker, out=None):
    if s.stride != 1 or s.pad != 0:
        return B.conv_fwd_ex(In, Ker, s.stride, s.pad, out=out)
    return (B.conv_fwd_bf16 if s.dtype == "bf16" else B.conv_fwd)(In, Ker, out=out)


def norm_err(out, ref):
    return float(np.linalg.norm(out.double().cpu().numpy() - ref) / np.linalg.norm(ref))


# One layer per compiled instance, with a tail of channels in its last chunk
# (the one-chunk instances, and 56 with bf16 Out: a tail in the only one).
PER_INSTANCE = {
    1: ConvShape("sp_i1", 12, 61, 35, 49, 62, 3, 3, "f32", 801, 1, 1),
    2: ConvShape("sp_i2", 7, 52, 465, 19, 23, 3, 3, "f32", 802, 1, 1),
    3: ConvShape("sp_i3", 16, 50, 75, 36, 43, 3, 3, "f32", 803),
    4: ConvShape("sp_i4", 1, 90, 72, 137, 158, 3, 3, "f32", 804, 2, 1),
    5: ConvShape("sp_i5", 19, 29, 12, 75, 74, 3, 3, "f32", 805, 2, 0),
    7: ConvShape("sp_i7", 27, 77, 12, 38, 37, 3, 3, "f32", 807),
    8: ConvShape("sp_i8", 29, 66, 14, 28, 26, 3, 3, "f32", 808, 1, 1),
    9: ConvShape("sp_i9", 7, 182, 6, 6, 5, 3, 3, "f32", 809, 2, 1),
    10: ConvShape("sp_i10", 5, 33, 38, 61, 59, 3, 3, "f32", 810, 1, 1),
    11: ConvShape("sp_i11", 1, 33, 33, 129, 124, 3, 3, "f32", 811, 2, 1),
    15: ConvShape("sp_i15", 4, 169, 687, 25, 29, 1, 1, "f32", 815),
    16: ConvShape("sp_i16", 26, 117, 5, 33, 37, 1, 1, "f32", 816),
    17: ConvShape("sp_i17", 1, 238, 10, 8, 6, 1, 1, "f32", 817, 2, 0),
    18: ConvShape("sp_i18", 21, 22, 10, 58, 46, 3, 3, "f32", 818, 2, 1),
    21: ConvShape("sp_i21", 1, 3, 6, 11, 11, 7, 7, "f32", 821, 2, 3),
    22: ConvShape("sp_i22", 2, 3, 184, 63, 77, 7, 7, "f32", 822, 2, 0),
    25: ConvShape("sp_i25", 10, 3, 26, 7, 5, 3, 3, "f32", 825, 2, 0),
    26: ConvShape("sp_i26", 20, 3, 7, 101, 127, 3, 3, "f32", 826, 2, 0),
    31: ConvShape("sp_i31", 27, 328, 553, 15, 15, 1, 1, "f32", 831),
    51: ConvShape("sp_i51", 7, 35, 7, 76, 78, 3, 3, "bf16", 851),
    52: ConvShape("sp_i52", 9, 35, 9, 83, 76, 3, 3, "bf16", 852),
    54: ConvShape("sp_i54", 29, 41, 306, 5, 4, 3, 3, "bf16", 854),
    55: ConvShape("sp_i55", 1, 35, 69, 132, 131, 3, 3, "bf16", 855),
    56: ConvShape("sp_i56", 9, 1, 93, 35, 45, 3, 3, "bf16", 856),
    57: ConvShape("sp_i57", 5, 74, 6, 54, 65, 3, 3, "bf16", 857),
    58: ConvShape("sp_i58", 1, 73, 14, 5, 5, 3, 3, "bf16", 858),
    59: ConvShape("sp_i59", 14, 176, 5, 13, 16, 1, 1, "bf16", 859),
    60: ConvShape("sp_i60", 3, 83, 5, 119, 152, 1, 1, "bf16", 860),
    61: ConvShape("sp_i61", 1, 31, 7, 5, 5, 5, 5, "bf16", 861),
    65: ConvShape("sp_i65", 26, 1, 36, 54, 60, 3, 3, "bf16", 865),
    66: ConvShape("sp_i66", 2, 3, 5, 96, 114, 3, 3, "bf16", 866),
}


def test_every_instance_has_a_layer():
    table = open(os.path.join(os.path.dirname(B.LIB_PATH), "csrc", "split_instances.inc")).read()
    assert {int(i) for i in re.findall(r"SPLIT_(?:F32|BF16)\((\d+),", table)} == set(PER_INSTANCE)
    for i, s in PER_INSTANCE.items():
        g = split_plan(s)
        assert g and g["id"] == i, (i, s, g)


GPU_SHAPES = EMULATED + SAMPLED + list(PER_INSTANCE.values()) + [
    ConvShape("sp_y18", 1, 512, 1024, 17, 17, 3, 3, "f32", 721, 1, 1),
    ConvShape("sp_f32_c48_k570", 2, 48, 570, 31, 31, 3, 3, "f32", 722),
    ConvShape("sp_f32_c144_93", 2, 144, 96, 93, 93, 3, 3, "f32", 723, 1, 1),
    ConvShape("sp_f32_c181", 23, 181, 92, 19, 19, 3, 3, "f32", 724),
    ConvShape("sp_f32_1x1_c165", 3, 165, 704, 120, 120, 1, 1, "f32", 725),
    ConvShape("sp_bf16_s2_c33", 2, 33, 13, 62, 77, 3, 3, "bf16", 739, 2, 0),
    ConvShape("sp_f32_image_7x7", 5, 3, 64, 131, 131, 7, 7, "f32", 726, 2, 3),
    ConvShape("sp_bf16_c288_1x1", 7, 288, 176, 79, 79, 1, 1, "bf16", 731),
    ConvShape("sp_bf16_c128", 32, 128, 128, 28, 28, 3, 3, "bf16", 732, 1, 1),
    ConvShape("sp_bf16_c144_k960", 3, 144, 960, 10, 10, 3, 3, "bf16", 733),
    ConvShape("sp_bf16_c16_k792", 4, 16, 792, 89, 89, 3, 3, "bf16", 734),
    ConvShape("sp_bf16_c832", 2, 832, 32, 58, 58, 3, 3, "bf16", 735, 1, 1),
    ConvShape("sp_bf16_c32_136", 8, 32, 64, 136, 118, 3, 3, "bf16", 736),
    ConvShape("sp_bf16_one_px", 2, 9, 20, 3, 3, 3, 3, "bf16", 737),
    ConvShape("sp_bf16_5x5", 2, 24, 40, 14, 12, 5, 5, "bf16", 738),
]


def plan_output(s, In, Ker):
    """The layer on a tile plan: a strided or padded one as the stride-1 problem
    over its phase images (image (a, b) of a channel is its padded rows a, a +
    stride, ... and columns b, b + stride, ...; tap (r, s) of the phase kernels
    is tap (r stride + a, s stride + b), zero past the last)."""
    st, pd = s.stride, s.pad
    if st == 1 and pd == 0:
        return B.conv_fwd_with_plan(In, Ker, B.conv_fwd_plan(*s.key()))
    inner = B.conv_fwd_ex_inner_shape(*s.key(), st, pd)
    C2, H2, W2, R2, S2 = inner[1], *inner[3:7]
    na, nb = min(st, s.R), min(st, s.S)
    assert C2 == s.C * na * nb
    X = torch.zeros(s.N, s.C, H2 * st, W2 * st, device=In.device)
    h, w = min(H2 * st, s.H + 2 * pd), min(W2 * st, s.W + 2 * pd)
    X[:, :, :h, :w] = torch.nn.functional.pad(In, (pd,) * 4)[:, :, :h, :w]
    Y = torch.zeros(s.K, s.C, R2 * st, S2 * st, device=In.device)
    Y[:, :, :s.R, :s.S] = Ker

    def phases(t, a, b):  # [.., C, rows, columns] of the na x nb images
        return torch.stack([t[:, :, i::st, j::st] for i in range(a) for j in range(b)], 2).flatten(1, 2).contiguous()
    X, Y = phases(X, na, nb), phases(Y, na, nb)
    assert X.shape == (s.N, C2, H2, W2) and Y.shape == (s.K, C2, R2, S2)
    return B.conv_fwd_with_plan(X, Y, B.conv_fwd_plan(*inner[:7]))


@pytest.mark.gpu
@pytest.mark.parametrize("s", GPU_SHAPES, ids=lambda s: s.name)
def test_parity(s):
    """Every output against the oracle, poisoned Out with guards, two runs
    equal; fp32: no further from the oracle than the tile plan."""
    g = split_plan(s)
    assert g, "on its tile plan"
    In, Ker = make_inputs(s)
    In_d, Ker_d = In.to(DEV), Ker.to(DEV)
    n = s.N * s.K * s.P * s.Q
    buf = torch.full((n + 128,), float("nan"), device=DEV)
    buf[:64] = buf[-64:] = 7.0
    out = buf[64:64 + n].view(s.N, s.K, s.P, s.Q)
    say(f"[gpu] split {s.name} id={g['id']} tile={g['tr']}x{g['tw']} co={g['co']} wgs={g['num_tiles']}")
    run(s, In_d, Ker_d, out)
    first = out.clone()
    run(s, In_d, Ker_d, out)
    torch.cuda.synchronize()
    assert torch.equal(first, out) and (buf[:64] == 7.0).all() and (buf[-64:] == 7.0).all()
    ref = oracle(s, In, Ker)
    got = out.cpu().numpy()
    # fp32 sums: each product's and each sum's rounding is below 2^-22 of the largest partial sum
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.max(np.abs(ref))
    if s.dtype == "f32":
        plan = plan_output(s, In_d, Ker_d)
        torch.cuda.synchronize()
        assert norm_err(out, ref) <= norm_err(plan, ref)


@pytest.mark.gpu
@pytest.mark.parametrize("s", [s for s in PER_INSTANCE.values() if s.dtype == "bf16"], ids=lambda s: s.name)
def test_bf16_out_is_the_rounded_fp32_out(s):
    """Each bf16 instance's bf16 Out is its fp32 Out, rounded; every element is written."""
    In, Ker = (x.to(DEV) for x in make_inputs(s))
    out = torch.full((s.N, s.K, s.P, s.Q), float("nan"), device=DEV, dtype=torch.bfloat16)
    say(f"[gpu] bf16 out {s.name}")
    B.conv_fwd_bf16_out(In, Ker, out=out)
    ref = B.conv_fwd_bf16(In, Ker).bfloat16()
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


@pytest.mark.gpu
@pytest.mark.parametrize("s", [EMULATED[0], EMULATED[2], SAMPLED[0]], ids=lambda s: s.name)
def test_integers_are_exact(s):
    In, Ker = make_inputs(s, kind="int")
    out = run(s, In.to(DEV), Ker.to(DEV))
    torch.cuda.synchronize()
    assert np.array_equal(out.double().cpu().numpy(), oracle(s, In, Ker))


SPECIAL = [ConvShape("sp_nonfinite_f32", 8, 64, 64, 58, 58, 3, 3, "f32", 741),
           ConvShape("sp_nonfinite_bf16", 2, 40, 24, 9, 11, 3, 3, "bf16", 742),
           ConvShape("sp_nonfinite_image", 8, 3, 64, 224, 224, 7, 7, "f32", 743, 2, 3),
           ConvShape("sp_nonfinite_point", 1, 512, 8192, 17, 17, 1, 1, "f32", 744),
           # units past the last tap, channel groups, one chunk
           ConvShape("sp_nonfinite_s2_c16", 3, 16, 8, 138, 169, 3, 3, "f32", 745, 2, 1),
           ConvShape("sp_nonfinite_s2_c10", 19, 10, 180, 19, 22, 3, 3, "f32", 746, 2, 0),
           ConvShape("sp_nonfinite_groups", 1, 37, 6, 7, 8, 3, 3, "f32", 747, 1, 1),
           ConvShape("sp_nonfinite_image_3x3", 10, 3, 64, 194, 194, 3, 3, "f32", 748, 2, 1),
           ConvShape("sp_nonfinite_bf16_s2", 1, 3, 7, 56, 61, 3, 3, "bf16", 749, 2, 0),
           ConvShape("sp_nonfinite_bf16_5x5", 2, 24, 40, 14, 12, 5, 5, "bf16", 750),
           ConvShape("sp_nonfinite_bf16_c128", 4, 128, 128, 28, 28, 3, 3, "bf16", 752, 1, 1),
           ConvShape("sp_nonfinite_bf16_vec", 8, 32, 64, 136, 118, 3, 3, "bf16", 753)]


@pytest.mark.gpu
@pytest.mark.parametrize("s", SPECIAL, ids=lambda s: s.name)
def test_infinities_and_nans(s):
    """Outputs that infinities, NaNs or overflowing sums touch are what IEEE
    arithmetic gives; the others are unaffected."""
    assert split_plan(s)
    In, Ker = make_inputs(s)
    In[0, 0, 2, 2], In[0, 1, 4, 5], In[0, 2, 6, 6] = float("inf"), float("-inf"), float("nan")
    In[-1, 1, 3, 3] = 3e38
    Ker[3, 0] = 1.0  # exact in bf16: its lower parts are zero
    Ker[5, 1, 0, 0] = float("inf")
    say(f"[gpu] non-finite {s.name}")
    out = run(s, In.to(DEV), Ker.to(DEV))
    torch.cuda.synchronize()
    got = out.double().cpu()
    ref = torch.nn.functional.conv2d(In.double(), Ker.double(), stride=s.stride, padding=s.pad)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    big = ref.abs() > 3.3e38  # (an fp32 sum may overflow on the way there)
    inf = torch.isinf(ref)
    assert torch.equal(got[inf], ref[inf])
    fin = torch.isfinite(ref) & ~big
    assert torch.isfinite(got[fin]).all()
    small = fin & (ref.abs() < 1e30)
    assert (got[small] - ref[small]).abs().max() <= 1e-5 * ref[small].abs().max()


@pytest.mark.gpu
@pytest.mark.parametrize("s", list(PER_INSTANCE.values()), ids=lambda s: s.name)
def test_second_pass_of_every_instance(s):
    """An infinity, its negative and a NaN at the corners and in the middle;
    fp32: also sums of 2^100 everywhere, no further from the 64-bit result
    than the tile plan."""
    In, Ker = make_inputs(s)
    In[0, 0, s.H // 2, s.W // 2], In[-1, -1, 0, 0] = float("inf"), float("-inf")
    In[0, -1, -1, -1] = float("nan")
    say(f"[gpu] second pass {s.name}")
    out = run(s, In.to(DEV), Ker.to(DEV))
    torch.cuda.synchronize()
    got = out.double().cpu()
    ref = torch.nn.functional.conv2d(In.double(), Ker.double(), stride=s.stride, padding=s.pad)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    inf, fin = torch.isinf(ref), torch.isfinite(ref)
    assert torch.equal(got[inf], ref[inf])
    if fin.any():
        assert (got[fin] - ref[fin]).abs().max() <= 1e-5 * ref[fin].abs().max()
    if s.dtype == "f32":
        In, Ker = make_inputs(s)
        In_d, Ker_d = In.to(DEV) * 2.0 ** 50, Ker.to(DEV) * 2.0 ** 50
        out, plan = run(s, In_d, Ker_d), plan_output(s, In_d, Ker_d)
        torch.cuda.synchronize()
        ref = oracle(s, In, Ker)
        # (layers of few outputs scatter: three roundings of half a unit, 3 x 2^-24, are allowed to any)
        assert norm_err(out * 2.0 ** -100, ref) <= max(norm_err(plan * 2.0 ** -100, ref), 3 * 2.0 ** -24)


LARGE = [SPECIAL[0], SPECIAL[2], SPECIAL[3],
         ConvShape("sp_large_4608", 32, 512, 512, 9, 9, 3, 3, "f32", 754),
         ConvShape("sp_large_9216", 2, 1024, 256, 28, 28, 3, 3, "f32", 755)]


@pytest.mark.gpu
@pytest.mark.parametrize("s", LARGE, ids=lambda s: s.name)
def test_sums_beyond_the_scaled_range(s):
    """Sums above 2^80 leave the scaled range: no further from the 64-bit
    result than the tile plan (or, where that does not take the layer as it
    is, than the 5e-7 that the fp32 plans stay within)."""
    assert split_plan(s)
    In, Ker = make_inputs(s)
    In, Ker = In * 2.0 ** 50, Ker * 2.0 ** 50
    In_d, Ker_d = In.to(DEV), Ker.to(DEV)
    say(f"[gpu] large sums {s.name}")
    out = run(s, In_d, Ker_d)
    torch.cuda.synchronize()
    ref = torch.nn.functional.conv2d(In.double(), Ker.double(), stride=s.stride, padding=s.pad).numpy()
    bound = 5e-7
    if s.stride == 1 and s.pad == 0:
        plan = B.conv_fwd_with_plan(In_d, Ker_d, B.conv_fwd_plan(*s.key()))
        torch.cuda.synchronize()
        bound = norm_err(plan, ref)
    err = norm_err(out, ref)
    say(f"[gpu] {s.name} error {err:.2e} bound {bound:.2e}")
    assert err <= bound


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_time_of_inputs_that_are_not_finite(dtype):
    """An all-NaN input takes at most 8 times a finite one (measured: fp32 3.7
    times, bf16 as long)."""
    s = ConvShape("sp_nan_time", 32, 128, 128, 30, 30, 3, 3, dtype, 756)
    assert split_plan(s)
    In, Ker = (x.to(DEV) for x in make_inputs(s))
    out = torch.empty(s.N, s.K, s.P, s.Q, device=DEV)
    us = {}
    for what, x in (("finite", In), ("NaN", torch.full_like(In, float("nan")))):
        run(s, x, Ker, out)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            run(s, x, Ker, out)
        b.record()
        torch.cuda.synchronize()
        us[what] = a.elapsed_time(b) * 100
    say(f"[gpu] {s.name} {dtype} {us}")
    assert torch.isnan(out).all()
    assert us["NaN"] <= 8 * us["finite"]


@pytest.mark.gpu
@pytest.mark.parametrize("scale_in,scale_ker", [(1e-30, 1e10), (1e-37, 1.0), (1e18, 1e18), (1e30, 1e-30), (2.0 ** -126, 2.0 ** 60)])
def test_extreme_magnitudes(scale_in, scale_ker):
    """The relative error does not depend on the operands' scale (the parts of
    an operand stay in bf16's normal range), also where sums leave the scaled
    range and are formed on the fp32 MFMA."""
    s = SPECIAL[0]
    In, Ker = make_inputs(s)
    In, Ker = In * scale_in, Ker * scale_ker
    out = run(s, In.to(DEV), Ker.to(DEV))
    torch.cuda.synchronize()
    ref = torch.nn.functional.conv2d(In.double(), Ker.double())
    assert ((out.double().cpu() - ref).norm() / ref.norm()).item() <= 5e-7


@pytest.mark.gpu
@pytest.mark.parametrize("s", [SAMPLED[0], EMULATED[0], SAMPLED[5], EMULATED[5]], ids=lambda s: s.name)
def test_unaligned_tensors(s):
    """In, Ker and Out one element past a 16-byte boundary."""
    In, Ker = make_inputs(s)
    ref = oracle(s, In, Ker)

    def shifted(x):
        b = torch.zeros(x.numel() + 8, dtype=x.dtype, device=DEV)
        v = b[1:1 + x.numel()].view(x.shape)
        v.copy_(x)
        return v
    out = shifted(torch.zeros(s.N, s.K, s.P, s.Q))
    run(s, shifted(In), shifted(Ker), out)
    torch.cuda.synchronize()
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))


@pytest.mark.gpu
def test_capture_and_side_streams():
    """Under graph capture conv_fwd runs the tile plan (no workspace is taken
    into the graph) and conv_fwd_ex_noalloc the split-operand kernels from its
    static scratch; replays between eager calls give the eager results."""
    s = SPECIAL[0]
    In, Ker = make_inputs(s)
    In_d, Ker_d = In.to(DEV), Ker.to(DEV)
    ref = oracle(s, In, Ker)
    a, b = (torch.zeros(s.N, s.K, s.P, s.Q, device=DEV) for _ in range(2))
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        B.conv_fwd(In_d, Ker_d, out=a)
        B.conv_fwd_ex_noalloc(In_d, Ker_d, out=b)
    st.synchronize()
    eager = a.clone()
    assert torch.equal(a, b)
    say("[gpu] capture")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        B.conv_fwd(In_d, Ker_d, out=a)
        B.conv_fwd_ex_noalloc(In_d, Ker_d, out=b)
    for _ in range(3):
        a.zero_()
        b.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(b, eager)
        assert np.max(np.abs(a.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
        other = B.conv_fwd(In_d, Ker_d)
        torch.cuda.synchronize()
        assert torch.equal(other, eager)


@pytest.mark.gpu
@pytest.mark.parametrize("s,bf16_out", [
    (ConvShape("sp_cap_bf16_s2", 8, 64, 128, 28, 28, 3, 3, "bf16", 761, 2, 1), False),
    (ConvShape("sp_cap_f32_s2", 32, 64, 128, 56, 56, 3, 3, "f32", 762, 2, 1), False),
    (ConvShape("sp_cap_bf16_5x5", 4, 64, 64, 24, 24, 5, 5, "bf16", 763), False),
    (ConvShape("sp_cap_bf16_out", 4, 128, 128, 30, 30, 3, 3, "bf16", 764), True),
], ids=lambda v: getattr(v, "name", None))
def test_capture_of_a_layer_whose_plan_needs_workspaces(s, bf16_out):
    """One eager call on a stream keeps the planned route's workspaces as well
    as the packed operand's, so the capture on that stream allocates nothing,
    and replays and eager calls in between agree."""
    assert split_plan(s), "layer is not on the split-operand route"
    In, Ker = make_inputs(s)
    In_d, Ker_d = In.to(DEV), Ker.to(DEV)
    ref = oracle(s, In, Ker)
    tol = 2.0 ** -8 if bf16_out else 1e-5  # bf16 Out: half a unit of 8 bits

    def call(out=None):
        if bf16_out:
            return B.conv_fwd_bf16_out(In_d, Ker_d, out=out)
        return B.conv_fwd_ex(In_d, Ker_d, s.stride, s.pad, out=out)

    def check(x):
        torch.cuda.synchronize()
        assert np.max(np.abs(x.float().cpu().numpy() - ref)) <= tol * np.max(np.abs(ref))

    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        out = call()
    check(out)
    say(f"[gpu] capture {s.name}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        call(out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        check(out)
        with torch.cuda.stream(st):
            other = call()
        check(other)
    B.release_workspaces(st)


@pytest.mark.gpu
@pytest.mark.parametrize("called_before", [True, False])
def test_a_captured_layer_outlives_a_larger_call(called_before):
    """Replays of a captured layer whose plan needs a workspace give the eager
    result after a larger layer has run on the stream, whether the layer's own
    workspace was kept at the capture or the graph allocates it."""
    s = ConvShape("sp_cap_small", 4, 64, 128, 28, 28, 3, 3, "bf16", 771, 2, 1)
    big = ConvShape("sp_cap_larger", 8, 64, 128, 60, 60, 3, 3, "bf16", 772, 2, 1)
    In, Ker = make_inputs(s)
    In_d, Ker_d = In.to(DEV), Ker.to(DEV)
    ref = oracle(s, In, Ker)
    bIn, bKer = (x.to(DEV) for x in make_inputs(big))
    st = torch.cuda.Stream()
    out = torch.zeros(s.N, s.K, s.P, s.Q, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        if called_before:
            B.conv_fwd_ex(In_d, Ker_d, s.stride, s.pad, out=out)
    st.synchronize()
    say(f"[gpu] capture {s.name} called_before={called_before}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        B.conv_fwd_ex(In_d, Ker_d, s.stride, s.pad, out=out)
    for _ in range(3):
        with torch.cuda.stream(st):
            B.conv_fwd_ex(bIn, bKer, big.stride, big.pad)
        torch.cuda.synchronize()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
    del graph
    torch.cuda.synchronize()
    B.release_workspaces(st)


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [(8, 128, 128, 30, 30, 3, 3), (1, 37, 64, 12, 12, 3, 3), (2, 64, 96, 40, 40, 1, 1)],
                         ids=str)
def test_tuned_layer_keeps_the_faster_route(dims):
    """After tuning, calls give the bits of the route that conv_fwd_split_plan
    reports: the split kernels', or the tuned plan's."""
    s = ConvShape("sp_tuned", *dims, "f32", 751)
    In, Ker = make_inputs(s)
    In_d, Ker_d = In.to(DEV), Ker.to(DEV)
    ref = oracle(s, In, Ker)
    before = split_plan(s)
    first = B.conv_fwd(In_d, Ker_d)
    say(f"[gpu] tune {dims}")
    out, plan, _ = B.conv_fwd_tune(In_d, Ker_d, top_n=24, reps=5)
    planned = B.conv_fwd_with_plan(In_d, Ker_d, plan)
    again = B.conv_fwd(In_d, Ker_d)
    torch.cuda.synchronize()
    for x in (out, planned, again):
        assert np.max(np.abs(x.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
    after = split_plan(s)
    say(f"[gpu] tuned {dims}: split before {bool(before)} after {bool(after)}")
    if before is None:
        assert after is None
    else:
        assert not torch.equal(first, planned), "the routes give the same bits: nothing is told apart"
    assert torch.equal(again, first if after else planned)
