"""fp16 prefill kernels whose exponentials leave the type's range: the rows are repeated from exact maxima, however small the excess over 65504 and whatever
the values are (a zero column hides no infinity: zero times an infinity is no number)."""
import numpy as np
import pytest

from paper_2604_12452_amd import inputs
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,d_pool,d_sel,H,S", [(inputs.MODE_GQA, 128, 128, 4, 2), (inputs.MODE_MLA, 512, 64, 4, 1)])
@pytest.mark.parametrize("rise", [13.5, 13.9, 14.2, 20.0, 60.0])       # nats above the first entries: 4 + 16 binades, where 65504 lies, are 13.86
@pytest.mark.parametrize("zero_column", [False, True])
def test_exponentials_past_65504(oracle, mode, d_pool, d_sel, H, S, rise, zero_column):
    wl = inputs.Workload("range", B=1, L=300, H=H, S=S, d_pool=d_pool, d_sel=d_sel, g=4, w=512, dtype="f16", mode=mode, seed=3, n_q=1)
    print(f"[case] {wl} rise {rise}", flush=True)
    Q, POOL, SEL = (inputs.to_f64(x, "f16") for x in inputs.gen_all(wl))
    Q[:] = 0.0
    Q[..., -1] = 1.0                                     # the logit is the selected component's last column
    SEL[:] = 0.0
    SEL[0, 200, ..., -1] = rise
    if zero_column:
        POOL[..., 0] = 0.0
    arrays = [inputs.to_storage(x.astype(np.float32), "f16") for x in (Q, POOL, SEL)]
    run = hp.GpuRun(wl, *arrays)
    run.dense()
    rows = np.arange(wl.L, dtype=np.int32)
    hp.check_dense(oracle, wl, run, rows, *(inputs.to_f64(a, "f16") for a in arrays))


@pytest.mark.parametrize("dtype,rise", [("f16", 14.5), ("f16", 30.0), ("f16", 85.0), ("f16", 95.0), ("bf16", 65.0), ("bf16", 85.0), ("bf16", 95.0)])
@pytest.mark.parametrize("w", [40, 300])
def test_gqa_repeats_from_row_sums(oracle, dtype, rise, w):
    """Rows that end beyond the limit are repeated from the logarithm of their sum where that is finite (a rise of up to 2^128, 88.7 nats), from
    exact maxima beyond.  w = 300: fp16 items whose references come from a sample of the tokens that all their rows see; w = 40: too few of those."""
    wl = inputs.Workload("sums", B=1, L=700, H=6, S=2, d_pool=128, d_sel=128, g=16, w=w, dtype=dtype, mode=inputs.MODE_GQA, seed=5)
    print(f"[case] {wl} rise {rise}", flush=True)
    Q, POOL, SEL = (inputs.to_f64(x, dtype) for x in inputs.gen_all(wl))
    Q[..., -1] = 1.0
    SEL[..., -1] = 0.0
    SEL[0, (70, 333, 651), ..., -1] = rise
    Q, POOL, SEL = (inputs.to_storage(x.astype(np.float32), dtype) for x in (Q, POOL, SEL))
    Qf, POOLf, SELf = (inputs.to_f64(x, dtype) for x in (Q, POOL, SEL))
    run = hp.GpuRun(wl, Q, POOL, SEL).condense()
    ref, differ = hp.check_condense(oracle, wl, run, Qf[:, wl.L - wl.nq:], POOLf, SELf)
    rows = np.arange(wl.L, dtype=np.int32)
    run.prefill()
    hp.check_prefill(oracle, wl, run, rows, Qf, POOLf, SELf, ref, differ)
    run.dense()
    hp.check_dense(oracle, wl, run, rows, Qf, POOLf, SELf)


@pytest.mark.parametrize("B,H", [(1, 4), (3, 16)])                    # pairs of wavefronts per 32 rows; one
@pytest.mark.parametrize("rise", [13.5, 14.5, 16.3, 17.0, 18.5, 30.0])   # nats: 65504 lies 4 + 16 binades (13.9) above the first entries
def test_mla_references_of_few_representatives(oracle, B, H, rise):
    """Rows whose reference comes from 1 to 15 representatives: whatever rises past the room above the largest of them is repeated."""
    wl = inputs.Workload("few", B=B, L=700, H=H, S=1, d_pool=512, d_sel=64, g=16, w=300, dtype="f16", mode=inputs.MODE_MLA, seed=6)
    print(f"[case] {wl} rise {rise}", flush=True)
    Q, POOL, SEL = (inputs.to_f64(x, "f16") for x in inputs.gen_all(wl))
    Q[..., -1] = 1.0
    SEL[..., -1] = 0.0
    SEL[:, (333, 651), ..., -1] = rise
    Q, POOL, SEL = (inputs.to_storage(x.astype(np.float32), "f16") for x in (Q, POOL, SEL))
    Qf, POOLf, SELf = (inputs.to_f64(x, "f16") for x in (Q, POOL, SEL))
    run = hp.GpuRun(wl, Q, POOL, SEL).condense()
    ref, differ = hp.check_condense(oracle, wl, run, Qf[:, wl.L - wl.nq:], POOLf, SELf)
    run.prefill()
    rows = np.arange(0, wl.L, 1 if B == 1 else 5, dtype=np.int32)
    hp.check_prefill(oracle, wl, run, rows, Qf[:, rows], POOLf, SELf, ref, differ)


@pytest.mark.parametrize("base,rise", [(2.0 ** 12, 24.0), (2.0 ** 12, 26.0), (2.0 ** 12, 40.0), (2.0 ** 13, 24.0), (2.0 ** 13, 32.0), (2.0 ** 13, 56.0)])
@pytest.mark.parametrize("w", [40, 300])
def test_gqa_repeats_where_a_reference_is_rounded_to_binades(oracle, base, rise, w):
    """Logits of 2^24 and 2^26 that rise by `rise` nats: the fp32 values a reference can take lie 2 and 8 binades apart there, more than a reference from row sums
    has room below 65504, so these rows are repeated from exact maxima."""
    wl = inputs.Workload("binades", B=1, L=700, H=6, S=2, d_pool=128, d_sel=128, g=16, w=w, dtype="f16", mode=inputs.MODE_GQA, seed=7)
    print(f"[case] {wl} base {base} rise {rise}", flush=True)
    Q, POOL, SEL = (inputs.to_f64(x, "f16") for x in inputs.gen_all(wl))
    Q[:] = 0.0
    Q[..., -1] = base
    Q[..., -2] = 1.0
    SEL[:] = 0.0
    SEL[..., -1] = base
    SEL[0, (71, 333, 651), ..., -2] = rise
    Q, POOL, SEL = (inputs.to_storage(x.astype(np.float32), "f16") for x in (Q, POOL, SEL))
    Qf, POOLf, SELf = (inputs.to_f64(x, "f16") for x in (Q, POOL, SEL))
    run = hp.GpuRun(wl, Q, POOL, SEL).condense()
    ref, differ = hp.check_condense(oracle, wl, run, Qf[:, wl.L - wl.nq:], POOLf, SELf)
    rows = np.arange(wl.L, dtype=np.int32)
    run.prefill(lse=False)
    hp.check_prefill(oracle, wl, run, rows, Qf, POOLf, SELf, ref, differ)
    run.dense(lse=False)
    hp.check_dense(oracle, wl, run, rows, Qf, POOLf, SELf)


@pytest.mark.parametrize("B,H,L,w", [(1, 4, 1300, 1024), (1, 4, 2300, 2048), (3, 16, 1300, 1024), (1, 16, 2300, 2048)])    # pairs of wavefronts per 32 rows, twice; one, twice
@pytest.mark.parametrize("above", [8.0, 10.5, 12.0, 12.5, 13.0, 14.0])        # nats
@pytest.mark.parametrize("value", [1.0, 0.1])
def test_mla_first_group_above_a_window_of_tokens(oracle, B, H, L, w, above, value):
    """The representative that fixes the reference of a row is the row's maximum, with a window of ordinary tokens far below it whose sum counts."""
    wl = inputs.Workload("sink", B=B, L=L, H=H, S=1, d_pool=512, d_sel=64, g=16, w=w, dtype="f16", mode=inputs.MODE_MLA, seed=8)
    print(f"[case] {wl} {above} nats, value {value}", flush=True)
    Q, POOL, SEL = (inputs.to_f64(x, "f16") for x in inputs.gen_all(wl))
    Q[:] = 0.0
    Q[..., -1] = 1.0
    SEL[:] = 0.0
    SEL[:, :16, ..., -1] = above
    POOL[:, :16] *= value
    Q, POOL, SEL = (inputs.to_storage(x.astype(np.float32), "f16") for x in (Q, POOL, SEL))
    Qf, POOLf, SELf = (inputs.to_f64(x, "f16") for x in (Q, POOL, SEL))
    run = hp.GpuRun(wl, Q, POOL, SEL).condense()
    ref, differ = hp.check_condense(oracle, wl, run, Qf[:, wl.L - wl.nq:], POOLf, SELf)
    run.prefill()
    rows = np.arange(w + 15, L, 9, dtype=np.int32)
    print("  rel err %.3e %.3e" % hp.check_prefill(oracle, wl, run, rows, Qf[:, rows], POOLf, SELf, ref, differ))


@pytest.mark.parametrize("L", [1024, 1025, 1130, 1300])               # items from row 1024 on take their references from a sample, also without representatives
@pytest.mark.parametrize("rise", [10.0, 14.5, 30.0, 95.0])
def test_gqa_references_around_the_first_sampled_item(oracle, L, rise):
    wl = inputs.Workload("from", B=1, L=L, H=4, S=2, d_pool=128, d_sel=128, g=16, w=2048, dtype="f16", mode=inputs.MODE_GQA, seed=9)
    print(f"[case] {wl} rise {rise}", flush=True)
    Q, POOL, SEL = (inputs.to_f64(x, "f16") for x in inputs.gen_all(wl))
    Q[..., -1] = 1.0
    SEL[..., -1] = 0.0
    SEL[0, (64, 517, L - 3), ..., -1] = rise                          # (64: one of the sample of the items from 1024 on; 517: of none)
    Q, POOL, SEL = (inputs.to_storage(x.astype(np.float32), "f16") for x in (Q, POOL, SEL))
    rows = np.arange(896, L, dtype=np.int32)
    run = hp.GpuRun(wl, Q, POOL, SEL).dense()
    Qf, POOLf, SELf = (inputs.to_f64(a, "f16") for a in (Q, POOL, SEL))
    hp.check_dense(oracle, wl, run, rows, Qf[:, rows], POOLf, SELf)
