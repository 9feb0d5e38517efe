"""Launch decisions, stream order and buffer extents of the library on a machine without a GPU: its host code is linked
against a HIP runtime that only records (launch_recorder.cpp), and the recorded launches are checked here."""
import json
import os
import re
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2510_03283_amd")


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    from paper_2510_03283_amd import build
    objs = [os.path.join(build.BUILD_DIR, s[:-4] + ".o") for s in build.sources()]
    if not all(os.path.exists(o) for o in objs):
        build.build_library()
    d = tmp_path_factory.mktemp("recorder")
    obj, exe = str(d / "recorder.o"), str(d / "recorder")
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-fPIE", "-std=c++17", "-O1", "-I", build.CSRC, "-c",
                    os.path.join(ROOT, "tests", "launch_recorder.cpp"), "-o", obj], check=True)
    subprocess.run(["g++", obj, *objs, "-o", exe], check=True)

    def run(call, **opts):
        args = [f"{k}={','.join(map(str, v)) if isinstance(v, (list, tuple)) else v}" for k, v in opts.items()]
        out = subprocess.run([exe, call, *args], capture_output=True, text=True, check=True).stdout
        return [json.loads(l) for l in out.splitlines()]

    return run


def status(rec):
    return next(r for r in rec if r["op"] == "return")


def plan(rec):
    return [r for r in rec if r["op"] == "plan"]


def slice_lifetimes(rec):
    """Every range of partial results: the launch that writes it, the launches that read it, and for each launch
    the number of launches of either stream it is known to follow (from stream order, event records and waits)."""
    n_done = [0, 0]                                   # launches issued per stream
    sees = [[0, 0], [0, 0]]                           # sees[s][t]: launches of t that whatever comes next on s follows
    events, live, out = {}, {}, []
    for i, r in enumerate(rec):
        if r["op"] == "record":
            s = r["stream"]
            events[r["event"]] = [n_done[t] if t == s else sees[s][t] for t in (0, 1)]
        elif r["op"] == "wait":
            s = r["stream"]
            sees[s] = [max(a, b) for a, b in zip(sees[s], events[r["event"]])]
        elif r["op"] == "launch":
            s = r["stream"]
            n_done[s] += 1
            sees[s][s] = n_done[s] - 1
            me = dict(i=i, kernel=r["kernel"], stream=s, at=n_done[s], follows=list(sees[s]))
            for kind, *rng in r["ranges"]:
                if kind == "parts_out":
                    life = dict(begin=rng[0], end=rng[0] + rng[1], writer=me, readers=[])
                    out.append(life)
                    live[tuple(rng)] = life
                elif kind == "parts_in":
                    assert tuple(rng) in live, f"launch {i} reads slices nobody wrote"
                    live[tuple(rng)]["readers"].append(me)
    return out


def check_slices(rec):
    def before(a, b):
        return b["follows"][a["stream"]] >= a["at"]
    lives = slice_lifetimes(rec)
    for n, x in enumerate(lives):
        assert x["readers"], f"slices of launch {x['writer']['i']} are never read"
        for r in x["readers"]:
            assert before(x["writer"], r), f"launch {r['i']} reads the slices of {x['writer']['i']} without an order between them"
        for y in lives[n + 1:]:
            if x["begin"] < y["end"] and y["begin"] < x["end"]:
                for a in [x["writer"], *x["readers"]]:
                    assert before(a, y["writer"]), (f"launch {y['writer']['i']} (stream {y['writer']['stream']}) overwrites slices of launch "
                                                    f"{x['writer']['i']} (stream {x['writer']['stream']}) that launch {a['i']} may still use")
    return lives


# Weight-gradient products are split between the caller's stream and the side stream by their sizes; where attention
# or the MLP is narrower than the model, both streams get some of them.
BWD = [
    dict(d=4096, hq=16, hkv=8, hd=128, F=1024, ft=[4096] * 4),
    dict(d=4096, hq=16, hkv=16, hd=128, F=512, ft=[4096] * 4),
    dict(d=2048, hq=16, hkv=16, hd=128, F=512, ft=[4096] * 8),
    dict(d=2560, hq=16, hkv=8, hd=128, F=9728, ft=[1640] * 8),
    dict(d=3584, hq=28, hkv=28, hd=64, F=9472, ft=[1200] * 8),
    dict(d=3072, hq=16, hkv=16, hd=128, F=8192, ft=[1600] * 8),
    dict(d=2048, hq=8, hkv=4, hd=128, F=5632, ft=[2048] * 8),
    dict(d=2048, hq=32, hkv=4, hd=64, F=5632, ft=[2048] * 8),
    dict(d=4096, hq=32, hkv=32, hd=128, F=11008, ft=[768] * 4),
]


@pytest.mark.parametrize("single_stream", [0, 1])
@pytest.mark.parametrize("lora", [0, 16])
@pytest.mark.parametrize("shape", BWD, ids=lambda s: f"d{s['d']}_q{s['hq'] * s['hd']}_F{s['F']}_{sum(s['ft'])}")
def test_slices_of_the_backward_do_not_meet(recorder, shape, lora, single_stream):
    rec = recorder("bwd", lora=lora, single_stream=single_stream, **shape)
    assert status(rec)["status"] == 0
    check_slices(rec)


def test_slices_of_the_backward_do_not_meet_over_a_range_of_shapes(recorder):
    both = 0
    for d in (1024, 2048, 4096):
        for qd in (512, 1024, 2048, 4096):
            for F in (512, 1024, 2816, 8192):
                for rows in (700, 2100, 9000, 17000, 33000):
                    rec = recorder("bwd", d=d, hq=qd // 128, hkv=qd // 128 // (2 if qd >= 256 else 1), hd=128, F=F, ft=[rows // 4 + i for i in range(4)], accumulate=1)
                    assert status(rec)["status"] == 0
                    both += len({x["writer"]["stream"] for x in check_slices(rec)}) == 2
    assert both > 20                                  # slices on both streams of one call do occur


@pytest.mark.parametrize("lora", [0, 16])
@pytest.mark.parametrize("shape", BWD + [dict(d=3584, hq=16, hkv=4, hd=128, F=2816, ft=[1412] * 8)],
                         ids=lambda s: f"d{s['d']}_q{s['hq'] * s['hd']}_F{s['F']}_{sum(s['ft'])}")
def test_one_stream_cuts_the_same_slices(recorder, shape, lora):
    """MACE_OPT_SINGLE_STREAM promises the same bits, so every product has the same tile and the same number of slices."""
    plans = []
    for single_stream in (0, 1):
        rec = recorder("bwd", lora=lora, single_stream=single_stream, **shape)
        assert status(rec)["status"] == 0
        check_slices(rec)
        plans.append([(r["name"], r["tile"], r["k_splits"]) for r in plan(rec)])
    assert plans[0] == plans[1]


@pytest.mark.parametrize("lora", [0, 16])
@pytest.mark.parametrize("single_stream", [0, 1])
def test_slices_of_the_forward_do_not_meet(recorder, lora, single_stream):
    n = 0
    for d, hq, hkv, F in ((1024, 8, 2, 2816), (2048, 8, 4, 5632), (4096, 32, 8, 11008)):
        for prefill, ft in (([300, 77], []), ([300], [500, 420]), ([], [700, 650]), ([1500] * 2, [900] * 4)):
            rec = recorder("fwd", d=d, hq=hq, hkv=hkv, hd=128, F=F, prefill=prefill, decode=[100, 40], ft=ft, lora=lora, single_stream=single_stream)
            assert status(rec)["status"] == 0
            n += len(check_slices(rec))
    assert n > 0


@pytest.mark.parametrize("rows", [80, 200, 400])
def test_two_pass_products_are_cut_as_fine_as_their_steps_allow(recorder, rows):
    """Both passes of a k tile are one step, so a reduction over 5632 has 88 of them: slices of eight are eleven, where twelve leave one empty."""
    rec = recorder("fwd", d=2048, hq=32, hkv=8, hd=64, F=5632, decode=[200] * 4, ft=[rows // 2] * 2)
    assert status(rec)["status"] == 0
    assert check_slices(rec)
    (down,) = [r for r in plan(rec) if r["k"] == 5632]
    assert down["k_splits"] == 11, down


@pytest.mark.parametrize("d,hq,hkv,hd,F", [(4096, 32, 32, 128, 11008), (2048, 32, 8, 64, 5632)])
def test_products_outside_the_four_wave_kernel_are_not_priced_as_its_tiles(recorder, d, hq, hkv, hd, F):
    """The adapter correction of dattn (bf16 output with a bf16 residual, K = 64) runs on the other kernel, whose tiles of 192 and 256 rows take
    two to three times as long there as four small ones: 36 - 59 us at 2255 x 4096, and the small ones are ahead at every number of rows."""
    for rows in (64, 700, 1622, 1833, 2044, 3521, 4154, 6053, 8800):
        rec = recorder("bwd", d=d, hq=hq, hkv=hkv, hd=hd, F=F, ft=[rows // 2, rows - rows // 2], lora=16)
        assert status(rec)["status"] == 0
        (r,) = [r for r in plan(rec) if r["name"] == "lora dattn gemm"]
        assert r["tile"] in ([64, 64], [64, 128]), (rows, r)


@pytest.mark.parametrize("hq,hkv,hd,ft,teams", [
    (32, 8, 64, [505, 470, 327, 400] * 2, 2), (32, 8, 64, [950, 941], 2), (32, 8, 64, [64] * 32, 2), (32, 8, 64, [134] * 24, 2),
    (32, 8, 64, [10] * 60, 1), (32, 8, 64, [30] * 40, 1), (32, 8, 64, [64] * 36, 1),          # many short sequences: more blocks than CUs
    (32, 8, 128, [396] * 8, 2), (32, 8, 128, [134] * 20, 2), (32, 32, 128, [396] * 2, 2), (32, 32, 128, [65] * 8, 2),
    (32, 8, 128, [10] * 60, 1), (32, 32, 128, [65] * 9, 1),
    (8, 8, 64, [60] * 16, 1), (32, 32, 128, [64] * 2, 1), (16, 8, 128, [64] * 16, 2),          # one query tile: nothing for a second team, but for a group of heads
    (8, 8, 64, [134] * 20, 2), (8, 8, 64, [396] * 8, 2),
    (32, 32, 64, [456] * 8, 1), (32, 32, 128, [1024] * 4, 1),
], ids=lambda v: f"{len(v)}x{v[0]}" if isinstance(v, list) else str(v))
def test_teams_of_the_attention_backward(recorder, hq, hkv, hd, ft, teams):
    """A block's second team of waves takes half of its turns where there are about as many blocks as CUs; past that, or without turns to share, it costs."""
    rec = recorder("bwd", d=512, hq=hq, hkv=hkv, hd=hd, F=512, ft=ft)
    assert status(rec)["status"] == 0
    (r,) = [r for r in rec if r["op"] == "launch" and "attn_bwd_dkdv_kernel" in r["kernel"]]
    assert f"ILi{hd}ELi{teams}E" in r["kernel"] and r["block"] == 256 * teams, r


def test_teams_of_the_checked_forms(recorder):
    """The GPU tests of the two forms run the form they name."""
    from test_gpu_attention_teams import FORMS, form_workload
    for form, teams in FORMS.items():
        rec = recorder("bwd", d=256, hq=form[0], hkv=form[1], hd=form[2], F=448, ft=[int(n) for n in form_workload(*form).batch.ft_lens])
        (r,) = [r for r in rec if r["op"] == "launch" and "attn_bwd_dkdv_kernel" in r["kernel"]]
        assert f"ELi{teams}E" in r["kernel"], (form, r)


MACE_BAD_SHAPE = -2


@pytest.mark.parametrize("rows", [1, 16, 33, 64, 65])
@pytest.mark.parametrize("weight", ["wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down"])
def test_misaligned_weights_are_refused(recorder, rows, weight):
    """A weight matrix that is not 16-byte aligned is refused on every path, the weight-streaming one for few rows included."""
    assert status(recorder("fwd", decode=[5] * rows))["status"] == 0
    r = status(recorder("fwd", decode=[5] * rows, misalign=weight))
    assert r["status"] == MACE_BAD_SHAPE, r


@pytest.mark.parametrize("rows", [1, 16, 33, 64, 65])
def test_misaligned_head_is_refused(recorder, rows):
    assert status(recorder("logits", decode=[5] * rows, n=rows))["status"] == 0
    r = status(recorder("logits", decode=[5] * rows, n=rows, misalign="w_lm"))
    assert r["status"] == MACE_BAD_SHAPE, r


def skinny_reads(rec):
    """Weight-streaming launches whose activations come in 16-row tiles: (pointer, bytes read, rows)."""
    out = []
    for r in rec:
        if r["op"] == "launch" and "skinny_kernelI" in r["kernel"]:
            mt, _, _, _, asrc, _ = re.search(r"skinny_kernelILi(\d+)ELi(\d+)ELi(\d+)ELb(\d)ELi(\d+)ELi(\d+)E", r["kernel"]).groups()
            if int(asrc) == 0:
                _, a, m, _, k = r["ranges"][0]
                out.append((a, int(mt) * 16 * k * 2, m))
    return out


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 31, 32, 33, 40, 47, 48, 49, 63, 64])
def test_few_row_products_read_inside_their_buffers(recorder, rows):
    # forward: the activation buffers hold whole 16-row tiles and lie one behind the other
    d, F = 1024, 2816
    rec = recorder("fwd", d=d, F=F, decode=[5] * rows)
    reads = skinny_reads(rec)
    assert len(reads) == (4 if rows > 16 else 3)
    for (_, n, m), k in zip(reads, [d] * (len(reads) - 1) + [F]):
        assert n == -(-m // 16) * 16 * k * 2, f"{m} rows of {k} values: {n} bytes read"
    # logits: the smallest workspace the call accepts
    lo, hi = 256, 1 << 24
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if status(recorder("logits", d=d, decode=[5] * rows, n=rows, work=mid))["status"] == 0 else (mid + 1, hi)
    rec = recorder("logits", d=d, decode=[5] * rows, n=rows, work=lo)
    work = next(r for r in rec if r["op"] == "work")
    (a, n, _), = skinny_reads(rec)
    assert work["ptr"] <= a and a + n <= work["ptr"] + lo, f"{rows} rows read {a + n - work['ptr'] - lo} bytes past a workspace of {lo}"


@pytest.mark.parametrize("rows", [1, 17, 63])
def test_fp32_logits_need_no_more_scratch_than_their_rows(recorder, rows):
    """fp32 models never take the few-row products, so their scratch holds the rows themselves and the head's bf16 form."""
    d, V = 1024, 4096
    work = -(-rows * d * 2 // 256) * 256 + V * d * 2
    rec = recorder("logits", d=d, V=V, bf16=0, decode=[5] * rows, n=rows, work=work)
    assert status(rec)["status"] == 0 and not skinny_reads(rec)


@pytest.mark.parametrize("d,hq,hkv,F,V", [(1024, 8, 8, 2816, 4096), (2048, 32, 8, 5632, 32000), (4096, 32, 32, 11008, 32000)])
@pytest.mark.parametrize("rows", [1, 17, 33, 64])
def test_plan_records_the_tiles_of_few_row_products(recorder, rows, d, hq, hkv, F, V):
    opts = dict(d=d, hq=hq, hkv=hkv, hd=d // hq, F=F, V=V, decode=[5] * rows)
    for rec in (recorder("fwd", **opts), recorder("logits", n=rows, **opts)):
        grids = [r["grid"][0] for r in rec if r["op"] == "launch" and "skinny_kernelI" in r["kernel"]]
        assert len(grids) == len(plan(rec)) > 0
        for g, r in zip(grids, plan(rec)):
            assert r["tile"] == [-(-rows // 16) * 16, r["n"] // g], (r, g)


def skinny_forms(rec):
    """Template arguments of the weight-streaming launches: row tiles, groups a block, ring slots, 8-row groups, source of the activations, epilogue, waves."""
    return [tuple(map(int, re.findall(r"L[ib](\d+)E", r["kernel"].split("skinny_kernelI")[1]))) for r in rec if r["op"] == "launch" and "skinny_kernelI" in r["kernel"]]


def test_groups_of_the_checked_few_row_products(recorder):
    """The GPU tests of the evenly shared groups run the forms that they name."""
    from test_gpu_skinny_even import FORMS
    F32, SWIGLU, QKV = 0, 1, 2
    for dims, by_rows in FORMS.items():
        opts = dict(zip(("d", "hq", "hkv", "hd", "F", "V"), dims))
        for rows, (qkv, gate_up, head) in by_rows.items():
            fwd, (last,) = (skinny_forms(recorder(call, n=rows, decode=[5] * rows, **opts)) for call in ("fwd", "logits"))
            tiles = -(-rows // 16) if rows <= 96 else 8
            got = {f[5]: f[:2] for f in fwd if f[5] != F32}
            if dims[4] <= 8192 or rows <= 96:
                assert got == {QKV: (tiles, qkv), SWIGLU: (tiles, gate_up)}, (dims, rows, fwd)
            assert last[:2] == (tiles, head) and last[5] == F32, (dims, rows, last)


def test_every_few_row_form_is_launched_by_some_batch(recorder):
    """A form of the kernel that nothing launches is not compiled."""
    from paper_2510_03283_amd import build
    names = subprocess.run(["nm", os.path.join(build.BUILD_DIR, "gemm_skinny.o")], capture_output=True, text=True, check=True).stdout
    compiled = {tuple(map(int, re.findall(r"L[ib](\d+)E", n))) for n in re.findall(r"skinny_kernelI(\S+)", names)}
    launched = set()
    for rows in (5, 17, 33, 49, 65, 81, 97):
        for d, hq, hkv, hd, F, V in ((320, 4, 4, 64, 704, 1024), (320, 64, 8, 128, 5120, 10240), (320, 64, 32, 128, 8192, 16384), (3072, 4, 4, 64, 14336, 4096), (1024, 32, 8, 64, 2752, 10304),
                                     (1024, 72, 36, 64, 4096, 12800), (1024, 50, 50, 128, 5504, 20800), (1024, 100, 50, 64, 7040, 32064), (1024, 256, 128, 64, 11008, 8192),
                                     (1024, 64, 32, 64, 5504, 8192), (4096, 64, 64, 64, 22016, 8192), (8192, 64, 32, 128, 5632, 32000)):
            opts = dict(d=d, hq=hq, hkv=hkv, hd=hd, F=F, V=V, n=rows, decode=[5] * rows)
            launched.update(skinny_forms(recorder("fwd", **opts)), skinny_forms(recorder("logits", **opts)))
    assert compiled - launched == set()


def test_blocks_of_few_row_products_share_their_groups_evenly(recorder):
    """A block takes its first group and its number of groups from the whole shares and the rest it is given, in 32 bits: together they are all groups once, and no block has more than its form holds."""
    n = 0
    for d, hq, hkv, hd, F, V in ((1024, 72, 36, 64, 11008, 10304), (2048, 32, 8, 64, 5632, 32000), (1024, 50, 50, 128, 7040, 12800), (4096, 32, 32, 128, 11008, 128256)):
        for rows in (1, 20, 40, 64, 80, 128):
            for call in ("fwd", "logits"):
                for r in recorder(call, d=d, hq=hq, hkv=hkv, hd=hd, F=F, V=V, n=rows, decode=[5] * rows):
                    if r["op"] != "launch" or "skinny_kernelI" not in r["kernel"]:
                        continue
                    _, nc, _, half, _, epi, _ = map(int, re.findall(r"L[ib](\d+)E", r["kernel"].split("skinny_kernelI")[1]))
                    (_, _, _, N, _), (_, share, rest) = r["ranges"]
                    groups, blocks = N // (8 if epi == 1 or half else 16), r["grid"][0]
                    b = np.arange(blocks, dtype=np.int64)
                    assert 0 <= rest < blocks and (b * rest < 2 ** 32).all()
                    first = b * share + b * rest // blocks
                    own = share + (b * rest % blocks + rest >= blocks)
                    assert first[0] == 0 and (first + own == np.append(first[1:], groups)).all() and 1 <= own.min() and own.max() <= nc, (groups, blocks, r["kernel"])
                    n += rest > 0
    assert n > 20


def test_tiles_of_the_checked_small_products(recorder):
    """The GPU tests of the small tiles run the tile that they name, with either output and any residual."""
    from test_gpu_small_tiles import SHAPES
    for (la, lb, M, N, K), tile in SHAPES.items():
        for out_bf16 in (0, 1):
            for resid in (0, 1, 2):
                (r,) = plan(recorder("product", la=la, lb=lb, M=M, N=N, K=K, ldc=N + 24, ldr=N + 2, out_bf16=out_bf16, resid=resid))
                assert tuple(r["tile"]) == tile, (la, lb, M, N, K, out_bf16, resid, r)


@pytest.mark.parametrize("groups", [[(300, 1, 2), (500, 2, 4)], [(256, 1, 1), (300, 2, 3), (700, 3, 5)], [(500, 2, 4), (300, 1, 2)]])
def test_slices_follow_their_row_group(recorder, groups):
    """The launcher starts row groups of more passes first; the slices of a group have to move with it."""
    r = status(recorder("gemm", groups=[v for g in groups for v in g], N=2048, K=4096))
    assert r["status"] == 0, r
    assert [g[1] for g in r["groups"]] == sorted((g[1] for g in groups), reverse=True)
    assert {tuple(g) for g in r["groups"]} == set(groups)


DECODE_HEADS = [(4096, 32, 32, 128), (2048, 32, 8, 64), (1024, 8, 2, 128), (1024, 8, 1, 64)]


@pytest.mark.parametrize("d,hq,hkv,hd", DECODE_HEADS, ids=lambda v: str(v))
@pytest.mark.parametrize("bf16", [0, 1])
def test_workspace_grows_with_requests_and_contexts(recorder, d, hq, hkv, hd, bf16):
    """What is enough for a batch is enough for one with fewer requests or shorter contexts, whatever tokens a block either takes.  (The requests'
    own rows only add: 66 rows and more, past the few-row products and their own scratch.)"""
    ns = [1, 2, 7, 16, 17, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 200, 255, 256, 257, 400]
    ctx = sorted({max(0, c + e) for c in (0, 128, 256, 384, 512, 640, 1024, 1536, 2048, 3072, 4096, 6144, 8192, 16384) for e in (-1, 0, 1)})
    rec = recorder("workspace", d=d, hq=hq, hkv=hkv, hd=hd, F=256, V=256, bf16=bf16, decode=ns, contexts=ctx, tokens=66)
    size = np.array([r["bytes"] for r in rec]).reshape(len(ns), len(ctx))
    assert size.min() > 0
    assert (np.diff(size, axis=0) >= 0).all() and (np.diff(size, axis=1) >= 0).all()


@pytest.mark.parametrize("rows,longest", [(1100, 4095), (1600, 4095), (2048, 4095), (2048, 1023)])
def test_shorter_contexts_fit_the_workspace_of_longer_ones(recorder, rows, longest):
    """64 requests of a 7B-class layer beside others, with adapters: the forward plans its scratch by the longest context that is there,
    the caller by the longest that may come."""
    opts = dict(d=4096, hq=32, hkv=32, hd=128, F=11008, V=32000)
    (size,) = recorder("workspace", decode=[64], contexts=[longest], tokens=rows - 64, **opts)
    for ctx in (longest, longest * 3 // 4, longest // 2, longest // 4, 511, 255, 127, 0):
        rec = recorder("fwd", prefill=[rows - 64], decode=[ctx] + [ctx // 2] * 63, lora=16, work=size["bytes"], **opts)
        assert status(rec)["status"] == 0, (ctx, status(rec))


@pytest.mark.parametrize("d,hq,hkv,hd,requests,context,splits", [
    (2048, 32, 8, 64, 1, 700, 6),          # a grid that leaves the chip idle: 128 tokens
    (2048, 32, 8, 64, 64, 400, 2),         # 256
    (2048, 32, 8, 64, 128, 400, 1),        # 2048 blocks of 256 take longer than 1024 of 512
    (2048, 32, 8, 64, 256, 800, 2),
    (2048, 32, 8, 64, 256, 120, 1),
    (4096, 32, 32, 128, 16, 400, 4),
    (4096, 32, 32, 128, 32, 800, 7),
    (4096, 32, 32, 128, 64, 4096, 5),      # a long stream: 1024
], ids=lambda v: str(v))
def test_decode_chunks_follow_the_work_of_the_grid(recorder, d, hq, hkv, hd, requests, context, splits):
    rec = recorder("fwd", d=d, hq=hq, hkv=hkv, hd=hd, F=1024, decode=[context] * requests)
    assert status(rec)["status"] == 0
    (grid,) = [r["grid"] for r in rec if r["op"] == "launch" and "attn_decode_kernel" in r["kernel"]]
    assert grid == [hkv, splits, requests]


# pi / 2 in three pieces of at most 32 bits and a rest (Machin's formula in integers)
PI_HALF = [3373259426 * 2.0 ** -31, 140128397 * 2.0 ** -61, 206333480 * 2.0 ** -91, 2.9038559739793605e-28]


def test_rotary_angles_have_fp64_accuracy(recorder):
    """The rotary sine and cosine against 80-bit results: three roundings of values up to 1 (the reduced angle, the
    polynomial, its last step) leave at most 3 * 2^-53; the result near a zero is as accurate as the reduced angle."""
    positions = [0, 1, 2, 3, 7, 100, 1023, 2047, 4095, 8191, 16383, 32768, 131071, 1 << 20, (1 << 24) + 1, (1 << 31) - 1] + list(range(5, 6000, 13))
    assert np.finfo(np.longdouble).eps < 2e-19
    rec = recorder("rope", positions=positions)
    assert len(rec) == 64 * len(positions)
    ang = np.array([r["angle"] for r in rec])
    k = np.rint(ang * (2 / np.pi)).astype(np.longdouble)
    # k has at most 31 bits: its product with a piece is exact in 64 bits of mantissa
    x = ang.astype(np.longdouble)
    for piece in PI_HALF:
        x = x - k * np.longdouble(piece)
    s, c = np.sin(x), np.cos(x)
    q = k.astype(np.int64) & 3
    sn = np.choose(q, [s, c, -s, -c])
    cs = np.choose(q, [c, -s, -c, s])
    for got, want in (([r["sin"] for r in rec], sn), ([r["cos"] for r in rec], cs)):
        err = np.abs(np.array(got).astype(np.longdouble) - want)
        print("largest error", float(err.max()))
        assert float(err.max()) <= 3 * 2.0 ** -53


@pytest.mark.parametrize("theta", [1e6, 1e4, 1.0, 1e-3, 1e-9, 1e-30, 1e-44])
def test_rotary_frequencies_stay_in_the_range_of_the_angles(recorder, theta):
    """Frequencies of bases down to the smallest mace_create accepts.  Up to 2^19 they are theta^(-2 i / hd); above (where
    the angle of a late position would leave the range of rope_sincos) whole turns are left out, to 64 bits of 2 pi."""
    f = np.array([r["value"] for r in recorder("create", theta=theta)])
    want = np.float64(np.float32(theta)) ** (-2.0 * np.arange(64) / 128)
    assert len(f) == 64 and f.max() <= 2.0 ** 19 and f.min() >= 0
    small = want <= 2.0 ** 19
    np.testing.assert_allclose(f[small], want[small], rtol=1e-15)      # (two libraries' pow, an ulp or two)
    if theta >= 1:
        assert small.all()
    two_pi = 4 * np.sum(np.array(PI_HALF, np.longdouble))
    turns = want[~small].astype(np.longdouble) / two_pi
    near = turns < 2.0 ** 40                                       # (whole turns of larger ones are below the last bit of theta's power)
    angle = (turns[near] - np.floor(turns[near])) * two_pi
    diff = np.abs(f[~small][near].astype(np.longdouble) - angle)
    assert np.all(np.minimum(diff, two_pi - diff) <= want[~small][near] * 2.0 ** -50)
