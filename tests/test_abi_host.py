"""Host half of the C ABI (no GPU needed): exports, metadata, work list, controller, errors."""
import json
import math
import os
import re

import numpy as np
import pytest

import _random_mixes as rm
from oracle import controller as oc
from oracle import meta as om
from paper_2609_38386_amd import dlfp as D
from paper_2609_38386_amd import workload as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    txt = open(os.path.join(ROOT, "include", "dlfp.h")).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b(?:int|const char\*)\s+(dlfp_\w+)\s*\(", txt)))


def test_library_exports_every_declared_symbol():
    L = D.lib()
    declared = _declared_functions()
    assert len(declared) >= 14
    for name in declared:
        assert hasattr(L, name), name
    assert set(declared) == set(D.EXPORTS)
    assert L.dlfp_version() == 100
    assert L.dlfp_status_string(-3) == b"capacity or workspace too small"


def _check_against_twin(dims, q_len, kv_len, bt, num_blocks, tuning=None):
    meta = D.dlfp_build_varlen_meta(dims, q_len, kv_len, bt, num_blocks, tuning)
    cu_q, q_pos0, slots = om.varlen_meta(q_len, kv_len, bt)
    n = len(q_len)
    assert meta.num_seqs == n and meta.num_tokens == cu_q[-1]
    assert meta.cu_q[:n + 1].tolist() == cu_q
    assert meta.q_pos0[:n].tolist() == q_pos0
    assert meta.slot_mapping[:meta.num_tokens].tolist() == slots
    om.check_work_list(meta.work, meta.num_prefill_units, q_len, kv_len, dims.num_q_heads,
                       dims.num_kv_heads, meta.num_groups, meta.workspace_bytes)
    om.check_append_records(meta.append_records, meta.work, meta.num_prefill_units, q_len,
                            kv_len, dims.num_kv_heads, meta.num_waiting_units)
    # decode units carry the block ids of their first two pages
    bt = np.asarray(bt)
    for u in meta.work[meta.num_prefill_units:]:
        s, kb, ke = int(u[0]), int(u[4]), int(u[5])
        pg = kb // 16
        assert u[14] == bt[s][pg]
        assert u[15] == (bt[s][pg + 1] if (ke - 1) // 16 >= pg + 1 else -1)
    return meta


def test_meta_tiny_iteration():
    cfg = wl.tiny_config()
    bt = wl.block_tables(cfg.seed, cfg.pages_per_seq(), cfg.pool_size())
    ctx = cfg.decoder_contexts()
    # block table rows: decoders first, then the prompt; batch order prompt first
    q_len = [128] + [1] * 4
    kv_len = [512] + [int(c) for c in ctx]
    rows = np.concatenate([bt[4:5], bt[:4]])
    dims = D.make_dims(16, 8)
    _check_against_twin(dims, q_len, kv_len, rows, cfg.pool_size())
    for tn in [D.dlfp_tuning(16, 64, 0), D.dlfp_tuning(32, 128, 0), D.dlfp_tuning(0, 0, 64),
               D.dlfp_tuning(0, 64, 0, 8)]:
        meta = _check_against_twin(dims, q_len, kv_len, rows, cfg.pool_size(), tn)
        if tn.decode_split_tokens == 16:
            assert meta.num_groups > 0
        if tn.prefill_tile_tokens == 8:   # 128 prompt tokens in tiles of 8, per KV head
            pre = meta.work[:meta.num_prefill_units]
            assert (pre[:, 3] <= 8).all() and len(np.unique(pre[:, 2])) == 16


@pytest.mark.parametrize("p,chunk", [(64, 0), (256, 17), (2048, 3)])
def test_meta_qwen3_0_6b_iterations(p, chunk):
    cfg = wl.qwen3_0_6b_config()
    bt = wl.block_tables(cfg.seed, cfg.pages_per_seq(), cfg.pool_size())
    its = cfg.iteration(p, chunk)
    q_len = [q for _, q, _ in its]
    kv_len = [k for _, _, k in its]
    rows = bt[[s for s, _, _ in its]]
    _check_against_twin(D.make_dims(16, 8), q_len, kv_len, rows, cfg.pool_size())


@pytest.mark.parametrize("seed", range(6))
def test_meta_random_mixes(seed):
    rng = np.random.default_rng(seed)
    g = [1, 2, 4, 8][seed % 4]
    hkv = int(rng.integers(1, 4))
    n = int(rng.integers(1, 7))
    q_len, kv_len = [], []
    for _ in range(n):
        if rng.random() < 0.5:
            q_len.append(1)
            kv_len.append(int(rng.integers(1, 300)))
        else:
            q = int(rng.integers(2, 200))
            q_len.append(q)
            kv_len.append(q + int(rng.integers(0, 300)))
    pages = [wl.pages_for(k) for k in kv_len]
    pool = sum(pages) + 5
    bt = wl.block_tables(seed, pages, pool, max_blocks=max(pages) + 2)
    tn = D.dlfp_tuning(int(rng.choice([0, 16, 48, 128])), int(rng.choice([0, 64, 192])), 0,
                       int(rng.integers(0, 128 // g + 1)))
    _check_against_twin(D.make_dims(g * hkv, hkv), q_len, kv_len, bt, pool, tn)


@pytest.mark.parametrize("i", range(rm.CASES))
def test_meta_of_the_random_gpu_mixes(i):
    """The random mixes the GPU parity test launches: the library's metadata equals
    the twin's, so every case's work list covers exactly the visible pairs before
    any of them runs on a device."""
    g, hkv, specs, tn, _, _ = rm.case(i)
    q_len, kv_len = [q for q, _ in specs], [k for _, k in specs]
    pages = [wl.pages_for(k) for k in kv_len]
    bt = wl.block_tables(rm.seed(i), pages, rm.pool(pages))
    _check_against_twin(D.make_dims(g * hkv, hkv), q_len, kv_len, bt, rm.pool(pages),
                        D.dlfp_tuning(*tn))


def test_meta_small_prefill_share_takes_latency_tiles():
    # a 32-token chunk over a 3000-token prefix next to one decoder (g = 2):
    # too few units at full tiles, so 16-token tiles and 256-key splits
    dims = D.make_dims(16, 8)
    q_len, kv_len = [32, 1], [3032, 2000]
    bt = np.arange(2 * 190, dtype=np.int32).reshape(2, 190)
    meta = _check_against_twin(dims, q_len, kv_len, bt, 2 * 190)
    pre = meta.work[:meta.num_prefill_units]
    assert meta.prefill_split_tokens == 256
    assert pre[:, 3].max() == 16 and len(pre) == 2 * 8 * 12
    # a 2048-token chunk fills the device at full tiles: throughput policy
    cfg = wl.qwen3_0_6b_config()
    bt6 = wl.block_tables(cfg.seed, cfg.pages_per_seq(), cfg.pool_size())
    its = cfg.iteration(2048, 3)
    meta = _check_against_twin(dims, [q for _, q, _ in its], [k for _, _, k in its],
                               bt6[[x for x, _, _ in its]], cfg.pool_size())
    assert meta.prefill_split_tokens >= 1024
    assert meta.work[:meta.num_prefill_units, 3].max() == 64


def test_meta_decode_tail_pieces_in_a_few_queue_rounds():
    # Qwen3-8B decoders alone (32 query / 8 KV heads): several queue rounds of
    # decode units, so each (sequence, KV head) range ends in a half and two
    # quarters of its last split part
    cfg = wl.qwen3_8b_config()
    pages = cfg.pages_per_seq()
    bt = wl.block_tables(cfg.seed, pages, int(sum(pages)))[:cfg.n_decoders]
    kv = [int(c) for c in cfg.decoder_contexts()]
    dims = D.make_dims(cfg.shape.num_q_heads, cfg.shape.num_kv_heads)
    meta = _check_against_twin(dims, [1] * len(kv), kv, bt, int(sum(pages)))
    split = meta.decode_split_tokens
    plain = sum(cfg.shape.num_kv_heads * math.ceil(k / split) for k in kv)
    assert meta.num_units > plain
    w = meta.work
    for s in range(3):
        rows = w[(w[:, 0] == s) & (w[:, 1] == 0)]
        rows = rows[np.argsort(rows[:, 4])]
        lens = rows[:, 5] - rows[:, 4]
        last = lens[-3:].sum()
        if last >= 64:
            assert lens[-3] >= lens[-2] >= lens[-1] and lens[-3] >= last // 2, lens
        assert (rows[:-3, 5] - rows[:-3, 4] == (rows[0, 5] - rows[0, 4])).all()


def test_meta_empty_batch():
    meta = D.dlfp_build_varlen_meta(D.make_dims(16, 8), [], [], np.zeros((0, 1), np.int32), 4)
    assert meta.num_seqs == 0 and meta.num_units == 0 and meta.workspace_bytes >= 256


@pytest.mark.parametrize("q", [1, 2])
def test_meta_longest_context(q):
    """The longest context an int32 holds (a pool of one block, repeated): the
    split policy's arithmetic stays in range and the units cover every key."""
    n = 2 ** 31 - 1
    bt = np.zeros((1, n // 16 + 1), dtype=np.int32)
    meta = D.dlfp_build_varlen_meta(D.make_dims(1, 1), [q], [n], bt, 1)
    units = meta.work
    assert meta.num_prefill_units == (0 if q == 1 else len(units))
    begin, end = np.sort(units[:, 4]), np.sort(units[:, 5])
    assert begin[0] == 0 and end[-1] == n and (begin[1:] == end[:-1]).all()


@pytest.mark.parametrize("hq,hkv,q_len,kv_len", [(64, 32, [1, 3821], [182, 26060]),
                                                 (64, 8, [1, 1, 3362], [3580, 1621, 3362]),
                                                 (16, 8, [1] * 32 + [256], [1280] * 32 + [4096])])
@pytest.mark.parametrize("resident", [0, 4096, 16384])
def test_meta_mixed_plans_fit_the_static_workspace(hq, hkv, q_len, kv_len, resident):
    """More wavefronts to fill make more splits, but never more partial results
    than the library's fixed workspace holds."""
    pages = [wl.pages_for(k) for k in kv_len]
    bt = wl.block_tables(1, pages, sum(pages))
    meta = D.dlfp_build_varlen_meta(D.make_dims(hq, hkv), q_len, kv_len, bt, sum(pages),
                                    D.dlfp_tuning(0, 0, resident))
    assert meta.workspace_bytes <= D.STATIC_WORKSPACE_BYTES


def _append_workgroups(records):
    """Workgroups of the one-launch form that write the append records; none above 128 records."""
    wgs = -(-records // 64) * 8
    return wgs if wgs <= 16 else 0


@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_meta_counts_the_append_workgroups_of_the_launch(g):
    """A page-aligned chunk of 256 tokens and 8 KV heads make 128 append records, 16
    workgroups of the launch: a plan of workgroup decode units leaves them their
    slots (512 workgroups are resident), so none ends between 496 and 512 units."""
    chunk, ctx = 256, 500
    dims = D.make_dims(8 * g, 8)
    for prefix in (0, 256):
        for decoders in range(20, 63):
            kv = [chunk + prefix] + [ctx] * decoders
            pages = [wl.pages_for(k) for k in kv]
            bt = np.zeros((len(kv), max(pages)), dtype=np.int32)
            m = D.dlfp_build_varlen_meta(dims, [chunk] + [1] * decoders, kv, bt, 1)
            assert m.num_append == 128
            fits = m.num_units + _append_workgroups(m.num_append) <= 512
            assert fits or m.num_units > 512, (g, prefix, decoders, m.num_units)


@pytest.mark.parametrize("g,decoders", [(2, [64, 100, 160, 256]), (1, list(range(512, 2048, 48))),
                                        (4, [2000, 9000]), (8, [300] * 8)])
def test_meta_decode_plan_is_the_decoders_own(g, decoders):
    """The decode share's plan depends on the decoders and on the slots that the
    prompt leaves, not on the prompt's keys: whole tiles of 32 rows are as many
    over any cached prefix, and the decode units beside them stay the same."""
    q = 64
    plans = []
    for prefix in (0, 512, 4096, 16384):
        kv = [q + prefix] + decoders
        bt = np.zeros((len(kv), max(wl.pages_for(k) for k in kv)), dtype=np.int32)
        m = D.dlfp_build_varlen_meta(D.make_dims(8 * g, 8), [q] + [1] * len(decoders), kv, bt, 1,
                                     D.dlfp_tuning(0, 32768, 0, 32 // g))
        plans.append((m.num_prefill_units, m.decode_split_tokens,
                      m.work[m.num_prefill_units:].tobytes()))
    assert all(p == plans[0] for p in plans), [p[:2] for p in plans]


@pytest.mark.parametrize("decoders,lo,hi", [(4, 10240, 38400), (8, 2816, 14336), (16, 1024, 6400),
                                            (28, 608, 4256)])
def test_meta_prefill_splits_leave_the_decode_share_its_slots(decoders, lo, hi):
    """A decode share that one round of wavefronts could hold is not crowded into
    the last few slots (units of 2500-3900 keys, one wavefront each) by prefill
    splits past one and a half units per compute unit."""
    prompts = [(900, 550), (560, 6800), (1100, 980)]
    kv = [q + p for q, p in prompts] + [lo + (hi - lo) * i // (decoders - 1)
                                        for i in range(decoders)]
    bt = np.zeros((len(kv), max(wl.pages_for(k) for k in kv)), dtype=np.int32)
    m = D.dlfp_build_varlen_meta(D.make_dims(16, 8), [q for q, _ in prompts] + [1] * decoders, kv,
                                 bt, 1)
    assert m.decode_split_tokens <= 2048, (m.num_prefill_units, m.decode_split_tokens)


@pytest.mark.parametrize("longest,reported", [(1, 16), (100, 112), (128, 128), (129, 144),
                                              (400, 400)])
def test_meta_decode_only_reports_the_longest_unit(longest, reported):
    """Without a prompt the launch chooses its kernel by the longest unit: many
    decoders that no split cuts report their longest context, in whole pages."""
    kv = [1 + (longest - 1) * i // 99 for i in range(100)]
    bt = np.zeros((100, wl.pages_for(longest)), dtype=np.int32)
    m = D.dlfp_build_varlen_meta(D.make_dims(16, 8), [1] * 100, kv, bt, 1)
    assert m.num_units == 800 and m.decode_split_tokens == reported


@pytest.mark.parametrize("decoders", [33, 35, 37, 40])
def test_meta_decode_only_units_even_over_the_compute_units(decoders):
    """Whole contexts of 33-40 decoders are 264-320 units for 256 compute units: a few
    of these would run two units of 1241 keys, so the contexts are cut."""
    bt = np.zeros((decoders, wl.pages_for(1241)), dtype=np.int32)
    m = D.dlfp_build_varlen_meta(D.make_dims(8, 8), [1] * decoders, [1241] * decoders, bt, 1)
    assert m.num_units >= 2 * 8 * decoders and m.work[:, 5].max() == 1241


def test_meta_prefill_splits_up_to_every_slot_stay_open():
    """Two units per compute unit leave no slot at all: the decode share then follows the
    prefill share on the whole device, in units cut for it."""
    prompts = [(125, 260), (86, 951), (89, 0), (132, 5), (81, 8065), (75, 898)]
    kv = [q + p for q, p in prompts] + [826 + 4377 * (2 * i + 1) // 30 for i in range(15)]
    bt = np.zeros((len(kv), max(wl.pages_for(k) for k in kv)), dtype=np.int32)
    m = D.dlfp_build_varlen_meta(D.make_dims(64, 8), [q for q, _ in prompts] + [1] * 15, kv, bt, 1)
    assert m.num_prefill_units == 512 and m.decode_split_tokens <= 512


def test_meta_errors():
    dims = D.make_dims(16, 8)
    bt = np.array([[0, 1, 2]], dtype=np.int32)
    with pytest.raises(D.DlfpError) as e:
        D.dlfp_build_varlen_meta(dims, [0], [5], bt, 4)
    assert e.value.status == -1
    with pytest.raises(D.DlfpError) as e:
        D.dlfp_build_varlen_meta(dims, [6], [5], bt, 4)
    assert e.value.status == -1
    with pytest.raises(D.DlfpError) as e:           # page 2 needs block 2, pool has 2 blocks
        D.dlfp_build_varlen_meta(dims, [1], [40], bt, 2)
    assert e.value.status == -2
    with pytest.raises(D.DlfpError) as e:           # 49 keys need 4 pages, table has 3
        D.dlfp_build_varlen_meta(dims, [1], [49], bt, 4)
    assert e.value.status == -2
    for bad in (D.make_dims(16, 8, head_dim=64), D.make_dims(16, 8, page_size=32),
                D.make_dims(12, 8), D.make_dims(128, 8)):
        with pytest.raises(D.DlfpError) as e:
            D.dlfp_build_varlen_meta(bad, [1], [5], bt, 4)
        assert e.value.status == -5
    with pytest.raises(D.DlfpError) as e:
        D.dlfp_build_varlen_meta(dims, [1], [5], bt, 4, D.dlfp_tuning(10, 0, 0))
    assert e.value.status == -1
    with pytest.raises(D.DlfpError) as e:           # g = 2: at most 64 tokens per tile
        D.dlfp_build_varlen_meta(dims, [1], [5], bt, 4, D.dlfp_tuning(0, 0, 0, 65))
    assert e.value.status == -1


def test_controller_worked_example_and_twin_agreement():
    with open(os.path.join(ROOT, "tests", "golden", "controller_observability.json")) as f:
        g = json.load(f)
    c = D.dlfp_controller_init(g["target_ms"], g["c_initial"], g["c_min"], g["c_max"],
                               g["quantum"])
    assert D.dlfp_controller_step(c, 3, True, g["observed_ms"]) == g["cap_after"]
    rng = np.random.default_rng(5)
    for trial in range(40):
        params = dict(target_ms=float(rng.uniform(5, 120)), c_initial=3072,
                      c_min=int(rng.choice([32, 128, 1024])), c_max=int(rng.choice([4096, 6144])),
                      quantum=128)
        cc = D.dlfp_controller_init(params["target_ms"], params["c_initial"], params["c_min"],
                                    params["c_max"], params["quantum"])
        twin = oc.Controller(params["target_ms"], params["c_initial"], params["c_min"],
                             params["c_max"], params["quantum"])
        for _ in range(50):
            ndec = int(rng.integers(0, 4))
            guarded = bool(rng.random() < 0.7)
            obs = float(rng.lognormal(math.log(params["target_ms"]), 0.8))
            assert D.dlfp_controller_step(cc, ndec, guarded, obs) == twin.step(ndec, guarded, obs)
            assert cc.cap == twin.cap


def test_controller_rejects_bad_observation_without_state_change():
    c = D.dlfp_controller_init(80.0, 3072, 1024, 6144)
    for bad in (0.0, -3.0, float("nan"), float("inf")):
        with pytest.raises(D.DlfpError) as e:
            D.dlfp_controller_step(c, 2, True, bad)
        assert e.value.status == -1
        assert c.cap == 3072
    # an unguarded step ignores the observation entirely
    assert D.dlfp_controller_step(c, 2, False, float("nan")) == 3072
    with pytest.raises(D.DlfpError):
        D.dlfp_controller_init(80.0, 512, 1024, 6144)
    with pytest.raises(D.DlfpError):
        D.dlfp_controller_init(float("nan"), 3072, 1024, 6144)


def test_stream_hold_rejects_out_of_range_durations_before_any_launch():
    for us in (0, -5, D.MAX_HOLD_US + 1):
        with pytest.raises(D.DlfpError) as e:
            D.dlfp_stream_hold(us, stream=0)
        assert e.value.status == -1


def test_grid_layout_and_decode_depth_policy():
    """Launches with both shares and more prefill units than compute units lead with
    one prefill unit per compute unit; otherwise every prefill unit comes first.
    Decode-only launches keep two pages in flight; the overrides are honoured."""
    dims = D.make_dims(64, 8)
    cfg = wl.qwen3_32b_config()
    pages = cfg.pages_per_seq()
    nb = int(sum(pages))
    bt_all = wl.block_tables(cfg.seed, pages, nb)
    for p, c, dec, pre in [(8192, 3, True, True), (512, 5, True, True), (8192, 3, False, True),
                           (512, 0, True, False)]:
        its = [x for x in cfg.iteration(p, c) if (x[1] > 1 and pre) or (x[1] == 1 and dec)]
        ql = [x[1] for x in its]
        kl = [x[2] for x in its]
        bt = bt_all[[x[0] for x in its]]
        m = D.dlfp_build_varlen_meta(dims, ql, kl, bt, nb)
        if dec and pre and m.num_prefill_units > 256:
            assert m.prefill_lead_units == 256
        else:
            assert m.prefill_lead_units == m.num_prefill_units
        assert m.decode_pages_in_flight == (2 if m.num_prefill_units == 0 else
                                            m.decode_pages_in_flight)
        assert m.decode_pages_in_flight in (1, 2)
        forced = D.dlfp_build_varlen_meta(dims, ql, kl, bt, nb,
                                          D.dlfp_tuning(0, 0, 0, 0, -1, 1))
        assert forced.prefill_lead_units == forced.num_prefill_units
        assert forced.decode_pages_in_flight == 1
    with pytest.raises(D.DlfpError):
        D.dlfp_build_varlen_meta(dims, ql, kl, bt, nb, D.dlfp_tuning(0, 0, 0, 0, 0, 3))


def test_probe_library_exports_its_declared_symbols():
    import ctypes
    txt = open(os.path.join(ROOT, "include", "dlfp_probe.h")).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    declared = sorted(set(re.findall(r"\bint\s+(dlfp_probe_\w+)\s*\(", txt)))
    assert declared == ["dlfp_probe_hbm_read", "dlfp_probe_mfma"]
    path = os.path.join(ROOT, "paper_2609_38386_amd", "libdlfp_probe.so")
    L = ctypes.CDLL(path)
    for name in declared:
        assert hasattr(L, name), name
