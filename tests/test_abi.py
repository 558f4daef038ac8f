"""The C-ABI library on a machine without a GPU: it loads, exports every symbol the header
declares, sizes buffers, and rejects bad arguments before touching the device."""
import ctypes as C
import math
import os
import re

import numpy as np
import pytest

import paper_2605_24786_amd as pkg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def clib():
    return pkg.load_library()


def test_exports_every_declared_symbol(clib):
    header = open(os.path.join(ROOT, "include", "conf_kv.h")).read()
    body = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(conf_kv_[a-z0-9_]+)\s*\(", body))
    assert declared == set(pkg.SYMBOLS), declared ^ set(pkg.SYMBOLS)
    for name in declared:
        assert getattr(clib, name) is not None


def test_config_struct_matches_header():
    header = open(os.path.join(ROOT, "include", "conf_kv.h")).read()
    block = re.search(r"typedef struct conf_kv_config \{(.*?)\} conf_kv_config;", header, re.S).group(1)
    block = re.sub(r"/\*.*?\*/", "", block, flags=re.S)
    names = []
    for decl in block.split(";"):
        decl = decl.strip()
        if not decl:
            continue
        decl = re.sub(r"^(const\s+)?(int32_t|uint64_t|float)\s*\*?", "", decl)
        names += [n.strip().lstrip("*") for n in decl.split(",")]
    assert names == [f[0] for f in pkg.ConfKVConfig._fields_]


def _cfg(**kw):
    base = dict(n_layers=2, batch=1, n_q_heads=8, n_kv_heads=2, head_dim=128, vocab=1000, capacity=256,
                fp16_window=16, protected_window=8, n_tight=[64, 64], n_loose=[128, 128])
    base.update(kw)
    return pkg.make_config(**base)


def test_buffer_sizes(clib):
    cfg, *_ = _cfg()
    sb, kb = clib.conf_kv_state_bytes(C.byref(cfg)), clib.conf_kv_scratch_bytes(C.byref(cfg))
    U, cap, D = 4, 256, 128
    payload = U * (cap * (2 * D + 4 + 8) + 32 * 2 * D * 2)      # INT8 rows + scales + meta + FP16 ring
    assert payload <= sb <= payload + 64 * 1024 and sb % 256 == 0 and kb > 0
    cfgc, *_ = _cfg(scale_mode="channel")                        # per-channel scales: [U][D], not [U][cap]
    sbc = clib.conf_kv_state_bytes(C.byref(cfgc))
    assert 0 < sbc < sb and sb - sbc >= U * (cap - D) * 4 - 4 * 256
    cfg16, *_ = _cfg(fp16_window=-1)                             # FP16-only: no INT8 planes
    sb16 = clib.conf_kv_state_bytes(C.byref(cfg16))
    assert U * cap * (4 * D + 8) <= sb16 <= U * cap * (4 * D + 8) + 64 * 1024


def test_prompt_phase_scratch(clib):
    """The prompt-phase kernels cut their work into parts only as far as the scratch that is there anyway holds them: the
    statistics of the longest prompt (12 bytes per row) or the two-launch form's scores, and the ranking arrays."""
    # (layers, batch, kv-heads, heads per kv-head, capacity): statistics are the larger one, then the scores
    for L, B, H, G, cap, mb in [(1, 1, 8, 16, 32768, 61.998), (1, 8, 8, 8, 32768, 438.049), (32, 1, 8, 16, 32768, 159.523)]:
        cfg, *_ = _cfg(n_layers=L, batch=B, n_q_heads=G * H, n_kv_heads=H, vocab=32000, capacity=cap, fp16_window=64,
                       n_tight=[cap // 4] * L, n_loose=[cap // 2] * L, max_chunk=2)
        assert clib.conf_kv_scratch_bytes(C.byref(cfg)) / 1e6 == pytest.approx(mb, abs=1e-3)
    have = getattr(clib, "_ZN6confkv22observe_scratch_floatsEiii")
    plan = getattr(clib, "_ZN6confkv19observe_plan_floatsEiiiiiimi")
    first = getattr(clib, "_ZN6confkv19observe_first_blockEiidd")
    have.restype = plan.restype = C.c_size_t
    have.argtypes, plan.argtypes = [C.c_int] * 3, [C.c_int] * 6 + [C.c_size_t, C.c_int]
    first.restype, first.argtypes = C.c_int, [C.c_int, C.c_int, C.c_double, C.c_double]
    cut = 0
    for units in (1, 2, 3, 8, 40, 64, 256, 384):
        for G in (1, 3, 4, 8, 16):
            for cap in (16, 64, 272, 1024, 4160, 32768, 524288):
                rows = units * G * cap
                assert have(units, G, cap) == 3 * rows
                for T in {1, 15, 65, cap // 7 + 1, cap // 2 + 1, cap - 1}:
                    if T > cap:
                        continue
                    for chan in (0, 1):
                        for room in (3 * rows, 3 * rows + 5000, 6 * rows, 1 << 40):
                            for b0 in {0, first(G, T, 0.9, 0.1)}:        # all rows, and those that count at lambda = 0.9
                                n = plan(units, G, T, b0, T // 3, chan, room, 256)
                                assert 3 * units * G * -(-T // 16) * 16 <= n <= room, (units, G, cap, T, b0, chan, room)
                                cut += n > 3 * units * G * -(-T // 16) * 16
    assert cut > 1000


def test_prompt_phase_rows_that_count(clib):
    """Rows ahead of the first block add less than half of the smallest number that fp32 holds to any slot, all together
    (gain times G heads times lambda^k summed over their distances k from the last token); a row more would not be left out.
    The parts of what is left fit their scratch."""
    first = getattr(clib, "_ZN6confkv19observe_first_blockEiidd")
    first.restype, first.argtypes = C.c_int, [C.c_int, C.c_int, C.c_double, C.c_double]
    plan = getattr(clib, "_ZN6confkv19observe_plan_floatsEiiiiiimi")
    plan.restype, plan.argtypes = C.c_size_t, [C.c_int] * 6 + [C.c_size_t, C.c_int]
    left_out = 0
    for G in (1, 3, 16):
        for T in (1, 16, 151, 1000, 1001, 1017, 3001, 32768, 524288):
            for lam in (0.0, 0.5, float(np.float32(0.9)), float(np.float32(0.999)), 1.0):
                for gain in (0.0, 1e-30, 1.0 - lam, 1.0, 1e6):
                    b0 = first(G, T, lam, gain)
                    assert 0 <= b0 < -(-T // 16) * G and b0 % G == 0
                    for chan in (0, 1):
                        for units in (1, 8, 64):
                            for room in (3 * units * G * -(-T // 16) * 16, 1 << 40):
                                assert plan(units, G, T, b0, T // 3, chan, room, 256) <= room
                    if lam == 1.0:
                        assert b0 == 0
                    elif 0.0 < lam and gain > 0.0:
                        tail = lambda k: math.log2(gain * G / (1.0 - lam)) + k * math.log2(lam)     # of all distances from k on
                        if b0:
                            assert tail(T - b0 // G * 16) <= -150.0
                            left_out += 1
                        if b0 // G < (T - 1) // 16:              # the next block of tokens reaches further
                            assert tail(T - (b0 // G + 1) * 16 - 1) > -150.0
    assert left_out > 50


def test_many_rows_splits_leave_room_for_a_second_call(clib):
    """Workgroups of a call of many rows wait for the unit's other splits, one per CU: two such calls side by side must not
    fill the chip with waiting ones.  Beyond the splits of 256 slots, up to eight, a call takes half of the CUs, or the number
    of its workgroups that can wait on an XCD of 32 CUs (kv/8 units, all splits but one) stays below 16."""
    splits = getattr(clib, "_ZN6confkv18attend_wide_splitsEiiiii")
    full = 0
    for kv in (1, 2, 4, 8, 12, 16, 24, 32, 64):
        for B in (1, 2, 3, 4, 5, 8, 16, 32, 64):
            for n in (1, 64, 191, 192, 400, 600, 1000, 2048, 2560, 5000, 30000):
                for most in (8, 16):
                    for major in {0, kv if kv % 8 == 0 else 0}:
                        units, ns = kv * B, splits(kv * B, major, n, most, 256)
                        plain = 1
                        while 2 * plain <= 8 and 2 * plain * units <= 256 and n // (2 * plain) >= 256:
                            plain *= 2
                        assert plain <= ns <= most and (ns == 1 or ns * units <= 256)
                        if ns > plain and 2 * ns * units > 256:
                            assert major and major // 8 * (ns - 1) < 16, (kv, B, n, most, ns)
                            full += 1
    assert full                                                  # (64 units of 8 kv-heads in four splits, 16 in sixteen)
    assert splits(16, 16, 2560, 16, 256) == 8 and splits(16, 8, 2560, 16, 256) == 16


def test_tiles_of_a_split(clib):
    """The bound on a split's tiles that decides whether the many-rows kernel can keep its probabilities: no split of a unit
    of at most n slots, with any number of FP16 slots up to n16, has more (INT8 slots cut at multiples of 32, FP16 slots evenly),
    and the bound is at most one too large.  Every count of FP16 slots, at lengths around the limits of 24 and 48 tiles."""
    bound = getattr(clib, "_ZN6confkv10rows_tilesEiiii")
    def need(n, ns):                                             # with any number of FP16 slots
        n16 = np.arange(min(n, max(windows)) + 1)
        n8, most = n - n16, np.zeros(len(n16), int)
        for j in range(ns):
            lo = n8 * j // ns & ~31
            hi = n8 if j == ns - 1 else n8 * (j + 1) // ns & ~31
            part16 = n16 * (j + 1) // ns - n16 * j // ns
            most = np.maximum(most, -(-(hi - lo) // 32) + -(-part16 // 16))
        return most

    windows = (0, 1, 15, 16, 17, 31, 32, 33, 48, 64, 79, 80, 112, 128, 144, 145, 300)
    at_limit = 0
    for ns in (1, 2, 3, 4, 8, 16):
        lengths = {*range(1, 300)}
        for tiles in (24, 48):
            lengths |= {*range(max(1, 32 * ns * (tiles - 1) - 40 * ns), 32 * ns * tiles + 2, 1 if ns <= 4 else 3)}
        for n in sorted(lengths):
            most = need(n, ns)
            for n16_ub in {min(w, n) for w in windows}:
                for least in {min(w, n16_ub) for w in (0, 5, 16, n16_ub)}:
                    top, got = most[least:n16_ub + 1].max(), bound(n, least, n16_ub, ns)
                    assert top <= got <= top + 1, (ns, n, least, n16_ub, got, top)
                    at_limit += got in (24, 48)
        for n in range(1, 32 * ns * 24, 7):
            for least in (0, 16):                                # what a shorter unit needs is there
                assert need(n, ns)[min(n, least):145].max() <= bound(n + 1, min(n + 1, least), min(n + 1, 144), ns), (ns, n, least)
                assert bound(n, min(n, least), min(n, 144), ns) <= bound(n + 40, min(n + 40, least), min(n + 40, 144), ns), (ns, n, least)
            assert bound(n, n, n, ns) == -(-(-(-n // ns)) // 16)   # FP16-only: no INT8 slots
    assert at_limit > 1000


def test_every_hook_is_in_the_header_and_read_once():
    """The environment variables of the library (those of trace builds aside): described in the header, and read when a handle
    is created or the first call planned, but for the one that the header says is read by each call."""
    header = open(os.path.join(ROOT, "include", "conf_kv.h")).read()
    csrc = os.path.join(ROOT, "paper_2605_24786_amd", "csrc")
    read = {}
    for name in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, name)).read()
        text = re.sub(r"#ifdef CONFKV_TRACE.*?#endif", "", text, flags=re.S)
        for m in re.finditer(r'getenv\("(\w+)"\)', text):
            read.setdefault(m.group(1), []).append((name, text[:m.start()]))
    assert read and all(re.search(rf"\b{hook}=", header) for hook in read), [h for h in read if h not in header]
    for hook, places in read.items():
        for name, before in places:
            # the function at the left margin that the call stands in
            inside = re.findall(r"^[a-z][\w *&:]*?(\w+)\(", before, flags=re.M)[-1]
            assert inside in ("conf_kv_create", "device_limits") or hook == "CONF_KV_COMPACT_PAIRED", (hook, name, inside)


def test_split_division_is_exact_for_every_slot_number(clib):
    """Slices are cut with a multiplier and a shift per launch: around multiples of every split count, up to the largest int."""
    divisor = getattr(clib, "_ZN6confkv13split_divisorEiPi")
    divisor.restype = C.c_uint32
    top = 2**31 - 1
    for ns in range(2, 65):
        shift = C.c_int(-1)
        mul = divisor(ns, C.byref(shift))
        near = {m * ns + d for m in {*range(70), *(2**b // ns for b in range(12, 31)), *range(top // ns - 70, top // ns + 1)} for d in (-1, 0, 1)}
        wrong = [x for x in sorted(near) if 0 <= x <= top and (x * mul >> 32) >> shift.value != x // ns]
        assert not wrong, (ns, wrong[0])


@pytest.mark.parametrize("bad", [dict(head_dim=96), dict(n_q_heads=34, n_kv_heads=2), dict(n_q_heads=18, n_kv_heads=2, head_dim=64), dict(n_q_heads=7),
                                 dict(capacity=100), dict(capacity=128), dict(vocab=1), dict(alpha=1.5),
                                 dict(n_tight=[200, 64]), dict(protected_window=-1), dict(n_layers=0),
                                 dict(ema_decay=-0.1), dict(mass_gain=float("nan")), dict(_ranker=2),
                                 dict(_rank_scope=-1), dict(_scale_mode=2), dict(max_chunk=-1), dict(max_chunk=33),
                                 dict(max_chunk=5, scale_mode="channel"),
                                 dict(max_chunk=2, head_dim=64), dict(max_chunk=70, n_tight=[64, 64], n_loose=[200, 200]),
                                 dict(scale_mode="channel", head_dim=64), dict(evict_page=-1), dict(evict_page=1025),
                                 dict(evict_page=64, protected_window=200, capacity=256),
                                 dict(scale_mode="channel", fp16_window=-1),
                                 # the paged layout: pages a power of two, only whole INT8 pages evictable, ...
                                 dict(layout="paged"), dict(layout="paged", evict_page=24),
                                 dict(layout="paged", evict_page=16, fp16_window=32, protected_window=16),
                                 dict(layout="paged", evict_page=16, fp16_window=-1),
                                 dict(layout="paged", evict_page=16, protected_window=16, n_q_heads=2),
                                 dict(layout="paged", evict_page=16, protected_window=16, rank_scope="layer"),
                                 dict(layout="paged", evict_page=16, protected_window=16, capacity=144),
                                 dict(_layout=2)])
def test_bad_configs_are_rejected(clib, bad):
    kw = dict(bad)
    if "n_layers" in kw:
        kw.update(n_tight=[], n_loose=[])
    raw = {k[1:]: kw.pop(k) for k in list(kw) if k.startswith("_")}    # enum fields set past the binding's names
    cfg, *_ = _cfg(**kw)
    for k, v in raw.items():
        setattr(cfg, k, v)
    assert clib.conf_kv_state_bytes(C.byref(cfg)) == 0
    h = C.c_void_p()
    assert clib.conf_kv_create(C.byref(h), C.byref(cfg), 256, 512) == pkg.binding.ERR_BAD_SHAPE
    assert not h.value


def test_null_and_misaligned_arguments(clib):
    cfg, *_ = _cfg()
    h = C.c_void_p()
    E = pkg.binding.ERR_INVALID_ARG
    assert clib.conf_kv_create(None, C.byref(cfg), 256, 512) == E
    assert clib.conf_kv_create(C.byref(h), C.byref(cfg), None, 512) == E
    assert clib.conf_kv_create(C.byref(h), C.byref(cfg), 257, 512) == E
    assert clib.conf_kv_destroy(None) == E
    assert clib.conf_kv_attend(None, 0, 16, 16, 16, 16, None) == E
    assert clib.conf_kv_step(None, 16, None, None, None) == E
    assert clib.conf_kv_evict_compact(None, None) == E
    assert clib.conf_kv_lengths(None, None, None) == E
    assert clib.conf_kv_last_hip_error(None) == 0
    # the bandwidth probe validates its arguments before anything is launched
    bad = pkg.binding.ERR_INVALID_ARG
    assert clib.conf_kv_probe_read(None, 1024, 256, 4, None) == bad
    assert clib.conf_kv_probe_read(256, 1000, 256, 4, None) == bad       # not a multiple of 16
    assert clib.conf_kv_probe_read(264, 1024, 256, 4, None) == bad       # misaligned source
    assert clib.conf_kv_probe_read(256, 1024, 256, 0, None) == bad
    for s in range(-7, 1):
        assert pkg.strerror(s) and pkg.strerror(s) != "unknown status"
    assert pkg.strerror(-99) == "unknown status"


def test_no_cpu_fallback():
    import torch
    if torch.cuda.is_available():
        pytest.skip("GPU present")
    with pytest.raises(RuntimeError, match="needs a GPU"):
        pkg.ConfKV(n_layers=1, batch=1, n_q_heads=1, n_kv_heads=1, head_dim=64, vocab=10, capacity=64,
                   fp16_window=-1, protected_window=2, n_tight=[8], n_loose=[16])


def test_pyramid_budgets_match_the_oracle(clib):
    """Host arithmetic, no GPU: the library's pyramidal schedule against the oracle's formula."""
    from oracle import confkv_oracle as O
    for n0, L, beta, n_min in [(256, 12, 0.5, 96), (128, 12, 0.5, 96), (4096, 64, 0.5, 96),
                               (2048, 32, 0.5, 96), (1000, 7, 0.3, 10), (512, 1, 0.5, 96), (100, 4, 1.0, 96)]:
        assert pkg.pyramid_budgets(n0, L, beta, n_min) == O.pyramid_geometric(n0, L, beta, n_min)
    out = (C.c_int32 * 4)()
    for bad in [(0, 4, 0.5, 96), (64, 0, 0.5, 96), (64, 4, 0.0, 96), (64, 4, 1.5, 96), (64, 4, 0.5, 0)]:
        assert clib.conf_kv_pyramid_budgets(*bad, out) == pkg.binding.ERR_INVALID_ARG
    assert clib.conf_kv_pyramid_budgets(64, 4, 0.5, 96, None) == pkg.binding.ERR_INVALID_ARG


@pytest.mark.parametrize("names", [("_cuda_getCurrentRawStream", "_cuda_getDevice"), ("_cuda_getDevice",), ()])
def test_stream_handle_with_and_without_the_private_calls(names):
    from types import SimpleNamespace as NS
    private = {"_cuda_getCurrentRawStream": lambda device: 100 + device, "_cuda_getDevice": lambda: 3}
    torch = NS(_C=NS(**{n: private[n] for n in names}),
               cuda=NS(current_stream=lambda: NS(cuda_stream=7)))
    assert pkg.binding._stream_getter(torch)() == (103 if len(names) == 2 else 7)
