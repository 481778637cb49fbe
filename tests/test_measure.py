"""Host logic of the measurement tools (no GPU): the counter summaries that
bench.py attaches to its line are computed from rocprofv3 CSV files; here
from small synthetic files whose figures are worked out by hand."""
import csv
import json
import os

import pytest

from paper_2608_13057_amd import measure, moe

GU = "void tempo::(anonymous namespace)::k_gemm_big_f8<true>(tempo::(anonymous namespace)::F8Args)"
COPY = "void at::native::vectorized_elementwise_kernel<4, at::native::AUnaryFunctor<float, float, float, " \
       "at::native::binary_internal::MulFunctor<float> >, std::array<char*, 2ul> >(int, ...)"


def _write(path, header, rows):
    os.makedirs(os.path.dirname(path), exist_ok=True)
    with open(path, "w", newline="") as fh:
        w = csv.writer(fh)
        w.writerow(header)
        w.writerows(rows)


def _counters(d, rows):
    _write(os.path.join(d, "run_counter_collection.csv"), ["Kernel_Name", "Counter_Name", "Counter_Value"], rows)


def _agent(d):
    _write(os.path.join(d, "run_agent_info.csv"), ["Name", "Num_Xcc", "Simd_Count", "Max_Engine_Clk_Fcompute"],
           [["gfx950", 8, 1024, 2400]])


def test_kernel_classification():
    assert measure._is_gateup(GU)
    assert measure._is_gateup("void tempo::(anonymous namespace)::k_gemm_big<true>(tempo::gemm::GemmArgs)")
    assert not measure._is_gateup("void tempo::(anonymous namespace)::k_gemm_big<false>(tempo::gemm::GemmArgs)")
    assert measure._is_gateup("void tempo::gemm::k_gemm<false, 64, true, false>(tempo::gemm::GemmArgs)")
    assert not measure._is_gateup("void tempo::gemm::k_gemm<false, 64, false, false>(tempo::gemm::GemmArgs)")
    for t in (0, 1, 2):
        w = "void tempo::(anonymous namespace)::k_gemm_wide<%d, %s>(tempo::(anonymous namespace)::WideArgs)"
        assert measure._is_gateup(w % (t, "true")) and not measure._is_gateup(w % (t, "false"))
    assert measure._is_copy(COPY) and not measure._is_copy(GU)


@pytest.mark.parametrize("dtype,T,S,H,I,m_tile,route,name", [
    ("bf16", 512, 18, 4096, 1536, 64, "stream", "k_gemm<false, 64, true, false>"),
    ("bf16", 4, 18, 4096, 1536, 64, "stream_split", "k_gemm<false, 64, true, false>"),
    ("fp8", 64, 18, 4096, 1536, 256, "stream_split", "k_gemm<true, 256, true, false>"),
    ("fp8mx", 64, 18, 1152, 1408, 256, "stream", "k_gemm<true, 256, true, true>"),
    ("bf16", 64, 18, 4096, 1536, 256, "big", "k_gemm_big<true>"),
    ("fp8mx", 8192, 18, 4096, 1536, 256, "big_f8", "k_gemm_big_f8<true>"),
    ("bf16", 8192, 18, 4096, 1536, 256, "wide", "k_gemm_wide<2, true>"),
    ("fp8", 8192, 18, 4096, 1536, 128, "wide", "k_gemm_wide<0, true>"),
    ("fp8mx", 8192, 18, 4096, 1536, 128, "wide", "k_gemm_wide<1, true>")])
def test_kernel_name_is_the_librarys_choice(dtype, T, S, H, I, m_tile, route, name):
    """The benchmark line names the kernel that the library itself says it
    launches for the shape (one rule, asked for, not written twice), and the
    counter summaries recognise that name."""
    shape = moe.MoEShape(T=T, K=8, E=128, S=S, H=H, I=I, m_tile=m_tile, dtype=dtype)
    assert measure.stage2_route(shape) == route
    full = measure.gateup_kernel_name(shape)
    assert full.endswith("::" + name) and measure._is_gateup(full)
    with pytest.raises(ValueError):
        measure.stage2_route(moe.MoEShape(T=T, K=8, E=128, S=S, H=H, I=I, m_tile=96, dtype=dtype))


@pytest.mark.parametrize("dtype,m_tile,rows,E,K,S,H,I,wide", [
    ("bf16", 64, 48, 128, 8, 18, 4096, 1536, False), ("bf16", 64, 64, 128, 8, 18, 4096, 1536, True),
    ("bf16", 64, 24, 256, 8, 36, 7168, 2048, False), ("bf16", 64, 48, 256, 8, 36, 7168, 2048, True),
    ("bf16", 64, 48, 64, 6, 12, 3072, 2048, False), ("bf16", 64, 80, 64, 6, 12, 3072, 2048, True),
    ("bf16", 128, 48, 128, 8, 18, 4096, 1536, False), ("bf16", 128, 80, 128, 8, 18, 4096, 1536, True),
    ("bf16", 256, 24, 64, 8, 12, 2048, 1408, True), ("bf16", 256, 512, 128, 8, 18, 4096, 1536, True),
    ("bf16", 256, 288, 96, 8, 12, 2048, 768, False), ("bf16", 256, 16, 128, 8, 18, 4096, 1536, False),
    ("fp8", 64, 12, 128, 8, 18, 4096, 1024, False), ("fp8", 64, 24, 128, 8, 18, 4096, 1024, True),
    ("fp8", 64, 8, 128, 8, 18, 4096, 1536, True), ("fp8", 64, 8, 256, 8, 36, 7168, 2048, False),
    ("fp8", 128, 12, 128, 8, 18, 4096, 1536, True), ("fp8", 128, 64, 128, 8, 20, 2048, 512, False),
    ("fp8mx", 64, 96, 64, 6, 10, 2048, 1408, False), ("fp8mx", 64, 48, 128, 8, 18, 4096, 1536, True),
    ("fp8mx", 64, 24, 256, 8, 36, 7168, 2048, False), ("fp8mx", 256, 64, 32, 4, 6, 4096, 384, False),
    ("fp8mx", 256, 32, 64, 4, 12, 7168, 384, False), ("fp8mx", 256, 64, 32, 4, 6, 2048, 640, True),
    ("fp8mx", 256, 64, 64, 6, 10, 5120, 896, True)])
def test_wide_tiles_only_where_they_were_measured_faster(dtype, m_tile, rows, E, K, S, H, I, wide):
    """Points on both sides of the lines of experts_wide_wanted."""
    shape = moe.MoEShape(T=rows * E // K, K=K, E=E, S=S, H=H, I=I, m_tile=m_tile, dtype=dtype)
    assert (measure.stage2_route(shape) == "wide") == wide


@pytest.mark.parametrize("dtype,m_tile,rows,E,K,S,H,I,whole", [
    ("bf16", 64, 2, 128, 8, 18, 4096, 1536, True), ("bf16", 64, 16, 32, 4, 5, 5120, 2048, False),
    ("bf16", 64, 8, 16, 2, 2, 7168, 2048, False), ("bf16", 64, 8, 256, 8, 36, 7168, 2048, True),
    ("bf16", 64, 8, 64, 4, 10, 3072, 1024, True), ("bf16", 64, 1, 64, 4, 10, 3072, 1024, False),
    ("bf16", 64, 8, 96, 8, 12, 1536, 768, True), ("bf16", 128, 24, 128, 8, 18, 4096, 1536, False),
    ("bf16", 128, 128, 64, 4, 10, 3072, 1024, False), ("bf16", 128, 24, 96, 6, 16, 1152, 768, True),
    ("fp8", 64, 4, 64, 4, 10, 3072, 1024, True), ("fp8", 64, 1, 32, 4, 5, 5120, 2048, False),
    ("fp8", 128, 24, 128, 8, 20, 2048, 512, True), ("fp8", 128, 24, 64, 4, 10, 3072, 1024, False), ("fp8", 256, 8, 128, 8, 18, 4096, 1536, False),
    ("fp8mx", 256, 16, 96, 6, 16, 1152, 640, True), ("fp8mx", 128, 64, 32, 4, 5, 5120, 2048, False)])
def test_items_stay_whole_only_where_that_was_measured_faster(dtype, m_tile, rows, E, K, S, H, I, whole):
    """Points on both sides of the lines of stream_whole_items."""
    shape = moe.MoEShape(T=rows * E // K, K=K, E=E, S=S, H=H, I=I, m_tile=m_tile, dtype=dtype)
    assert measure.stage2_route(shape) == ("stream" if whole else "stream_split")


def test_padding_tokens_do_not_choose_the_kernel():
    """A padded batch runs on the kernels of the batch it holds: padding
    tokens make no rows.  (Sizes on both sides of every line of the rules.)"""
    for dtype in ("bf16", "fp8", "fp8mx"):
        for m_tile in (64, 128, 192, 256):
            for E, K, S, H, I in ((128, 8, 18, 4096, 1536), (256, 8, 36, 7168, 2048), (64, 6, 10, 2048, 1408), (16, 2, 2, 7168, 384)):
                kw = dict(K=K, E=E, S=S, H=H, I=I, m_tile=m_tile, dtype=dtype)
                for Tv in (1, 4, 40, 130, 200, 400, 700, 1100, 1700, 3000, 6000, 9000):
                    route = measure.stage2_route(moe.MoEShape(T=Tv, **kw))
                    for T in (Tv + 1, 2 * Tv, 16 * Tv):
                        assert measure.stage2_route(moe.MoEShape(T=T, T_valid=Tv, **kw)) == route, (kw, Tv, T)


def test_mfma_summary_arithmetic(tmp_path):
    """Two dispatches: busy cycles 2e8 / 3e8, GRBM_GUI_ACTIVE (summed over 8
    XCDs) 3.2e6 / 4.8e6, MOPS 1e8 / 1e8, mean duration 200 us.  Mean busy
    2.5e8 over 4e6 / 8 = 5e5 dispatch cycles x 1024 SIMDs: 0.48828125;
    clock 5e5 cycles / 200 us = 2.5 GHz; executed 1e8 x 512 flops in 200 us:
    256 TFLOP/s."""
    pmc, kt = str(tmp_path / "pmc"), str(tmp_path / "kt")
    _counters(pmc, [[GU, "SQ_VALU_MFMA_BUSY_CYCLES", 2e8], [GU, "SQ_VALU_MFMA_BUSY_CYCLES", 3e8],
                    [GU, "GRBM_GUI_ACTIVE", 3.2e6], [GU, "GRBM_GUI_ACTIVE", 4.8e6],
                    [GU, "SQ_INSTS_VALU_MFMA_MOPS_F8", 1e8], [GU, "SQ_INSTS_VALU_MFMA_MOPS_F8", 1e8],
                    ["other", "GRBM_GUI_ACTIVE", 1.0]])
    _agent(pmc)
    _write(os.path.join(kt, "run_kernel_stats.csv"), ["Name", "Calls", "AverageNs", "MinNs", "MaxNs", "Percentage"],
           [[GU, 2, 200000.0, 190000.0, 210000.0, 50.0]])
    out = str(tmp_path / "m.md")

    class A:
        pass

    a = A()
    a.pmc_dir, a.trace_dir, a.workload, a.m_tile, a.out, a.command1, a.command2 = \
        pmc, kt, "qwen3_prefill_fp8mx", 256, out, "c1", "c2"
    assert measure._mfma(a) == 0
    line = [l for l in open(out) if l.startswith("mfma_json: ")][0]
    d = json.loads(line[len("mfma_json: "):])
    assert d["mfma_busy"] == pytest.approx(0.48828125)
    assert d["clock_ghz"] == pytest.approx(2.5)
    assert d["executed_tflops"] == pytest.approx(256.0)
    assert d["dispatches"] == 2 and d["source_hash"] == measure.gemm_source_hash()


def test_traffic_summary_scales_by_the_copy(tmp_path):
    """The gate/up kernel's FETCH_SIZE (KiB per dispatch) is scaled by what the
    counter reads for the 256 MiB copy: a copy reading 131072 KiB where
    262144 KiB were read gives 2.0, so 1000 KiB of the kernel are 2048000
    bytes; WRITE_SIZE of the copy reads its true 262144 KiB (factor 1)."""
    fe, wr = str(tmp_path / "fe"), str(tmp_path / "wr")
    _counters(fe, [[GU, "FETCH_SIZE", 1000.0], [GU, "FETCH_SIZE", 1000.0], [COPY, "FETCH_SIZE", 131072.0]])
    _counters(wr, [[GU, "WRITE_SIZE", 50.0], [COPY, "WRITE_SIZE", 262144.0]])
    out = str(tmp_path / "t.md")

    class A:
        pass

    a = A()
    a.fetch_dir, a.write_dir, a.workload, a.m_tile, a.out, a.command1, a.command2 = \
        fe, wr, "qwen3_prefill_fp8mx", 256, out, "c1", "c2"
    assert measure._traffic(a) == 0
    line = [l for l in open(out) if l.startswith("traffic_json: ")][0]
    d = json.loads(line[len("traffic_json: "):])
    assert d["copy_fetch_factor"] == pytest.approx(2.0) and d["copy_write_factor"] == pytest.approx(1.0)
    assert d["fetch_bytes"] == pytest.approx(2048000.0) and d["write_bytes"] == pytest.approx(51200.0)
    assert d["bytes_per_launch"] == pytest.approx(2099200.0)


def test_committed_summaries_match_their_sources():
    """Every committed counter summary names the stage-2 source hash it was
    taken with; bench.py drops figures whose hash differs."""
    for name, m in (("qwen3_prefill_fp8mx", 256), ("qwen3_prefill_bf16", 256)):
        d = measure.committed_mfma(name, m)
        if d is not None:
            assert d["source_hash"] == measure.gemm_source_hash()
    b, current = measure.committed_traffic("qwen3_decode_bf16", 64)
    assert b is None or b > 0


def test_fits_are_of_the_current_kernels(tmp_path, monkeypatch):
    """The fit that the benchmark line attaches is the committed one of the
    same shape, dtype and M-tile only while the stage-2 sources are those that
    were timed; a summary of rows from two builds belongs to neither."""
    from paper_2608_13057_amd import profile

    rows = [dict(scope=sc, G=G, n=n, N=G * n, tiles=G * -(-n // 64), t_us=20.0 + 5.0 * G + 0.1 * G * n, p10=1.0, p90=1.0,
                 source_hash=measure.gemm_source_hash())
            for sc in ("gemm", "block") for G in range(1, 9) for n in (1, 8, 64, 128, 512, 1024)]
    path = tmp_path / "stage4.md"
    monkeypatch.setattr(measure, "fit_path", lambda *a: str(path))

    def fit(rows):
        path.write_text(profile.markdown(rows, "t", "c"))
        return measure.committed_fit("qwen3", "bf16", 64)

    f = fit(rows)
    assert f is not None and f["scope"] == "gemm" and f["model"] == "Eq. 1" and f["a"] > 0
    assert fit([dict(r, source_hash="0" * 16) for r in rows]) is None
    assert fit([{k: v for k, v in r.items() if k != "source_hash"} for r in rows]) is None
    assert fit(rows[:-1] + [dict(rows[-1], source_hash="0" * 16)]) is None
