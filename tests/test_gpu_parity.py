"""GPU parity: the HIP path (through the C ABI) against the float64 oracle on the same
seeded inputs.  Logits are compared element by element; decisions are compared with the
oracle's verify stage run on the GPU's own logits, every mismatch classified."""
import dataclasses

import numpy as np
import pytest
import torch

import synth
from oracle import model as om
from oracle import verify as ov
from tests import harness as hz

pytestmark = pytest.mark.gpu


def small_bf16(**kw):
    base = dict(name="small-bf16", dtype="bf16", L=2, d=320, H=8, Hkv=2, hd=64, F=576, V=5000,
                B=3, S=150, tree="widths_2455", depth=4, q_std=2.5, q_T=0.8, T=0.8,
                top_p=0.9, top_k=24, ragged=True, random_gains=True, seed_base=4242)
    base.update(kw)
    return synth.Workload(**base)


def _check_tree(run, tol):
    """Logits of the forward-sampled sessions against the oracle's float64 forward;
    decisions of EVERY row of every session against the oracle's verify stage on the GPU's
    logits; the walk of every session from the GPU's decisions."""
    z_ref = hz.oracle_tree_logits(run)
    n1 = run.host_in["tokens"].shape[1]
    zg = np.stack([run.outs["logits_out"][b * n1:(b + 1) * n1].numpy() for b in run.sessions])
    err = hz.logits_rel_err(zg.astype(np.float64), z_ref)
    hz.log(f"logits max rel err {err.max():.3e} over {len(run.sessions)} sessions (tol {tol})")
    assert err.max() <= tol, err.max()
    rep = hz.check_tree_decisions(run)
    hz.log(f"decisions (all {run.host_in['tokens'].shape[0]} sessions): {rep}")
    info = hz.agreement_on_oracle_logits(run, z_ref)
    hz.log(f"informational, on the oracle's own logits: {info}")
    assert rep.ok(), str(rep)
    return err, rep


@pytest.mark.parametrize("seed", hz.parity_seeds(synth.get("tiny-fp32"), 10))
def test_tree_tiny_fp32_full_config(seed):
    """The tiny fp32 workload at its full size (2 layers, d=256, vocab 4096, 8-node tree),
    ten parity seeds."""
    w = synth.get("tiny-fp32")
    run = hz.run_tree(w, seed=seed)
    _check_tree(run, tol=1e-4)


@pytest.mark.parametrize("variant", [
    dict(),                                                    # hd 64, G 4, 16-node tree
    dict(hd=128, H=4, Hkv=1, d=256, tree="chain_sib", depth=6, sib=2, V=4100),
    dict(hd=128, H=8, Hkv=8, tree="chain", depth=9, B=2, S=64, ragged=False, V=2048),
    dict(hd=64, H=8, Hkv=2, tree="chain_sib", depth=8, sib=7, B=2, S=700, top_k=64),
    # 8 query heads per kv head under a 64-node tree: 520 query rows, two query groups
    dict(hd=64, H=16, Hkv=2, d=256, tree="chain_sib", depth=8, sib=7, B=2, S=300, top_k=32),
    dict(hd=128, H=8, Hkv=1, d=256, tree="chain_sib", depth=8, sib=7, B=3, S=200, V=3000),
    # 8 query heads under a 36-node tree: 296 rows in two query groups of 148, i.e. four
    # 32-row tiles and a 20-row remainder, which is a padded 32-row tile of its own
    dict(hd=64, H=16, Hkv=2, d=256, tree="chain_sib", depth=4, sib=8, B=2, S=1024, V=3000),
    dict(hd=128, H=16, Hkv=2, d=256, tree="chain_sib", depth=4, sib=8, B=2, S=600, V=3000),
])
def test_tree_small_bf16(variant):
    w = small_bf16(**variant)
    run = hz.run_tree(w)
    _check_tree(run, tol=2e-2)


@pytest.mark.parametrize("variant", [
    dict(),
    dict(hd=128, H=4, Hkv=1, d=256, tree="chain_sib", depth=6, sib=2, V=4112),
    dict(hd=64, H=16, Hkv=2, d=256, tree="chain_sib", depth=8, sib=7, B=2, S=300, top_k=32,
         V=4096),
])
def test_tree_small_bf16_packed_weights(variant):
    """The same forward with the dense matrices in the packed layout
    (acespec_pack_weight): every GEMM takes its weight operands straight from the packed
    copy."""
    w = small_bf16(**dict(dict(V=5008), **variant))
    run = hz.run_tree(w, packed=True)
    _check_tree(run, tol=2e-2)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("B, depth, d, F", [
    (1, 0, 320, 576), (1, 15, 320, 576), (1, 16, 1024, 2048), (3, 15, 320, 576),
    (7, 6, 320, 576), (1, 64, 1024, 2048), (5, 15, 320, 576), (7, 15, 320, 576),
    (9, 15, 1024, 2048), (5, 28, 320, 576), (9, 31, 1024, 2048), (17, 16, 320, 576),
    (17, 31, 320, 576), (5, 54, 2048, 4096)])
def test_tree_row_counts(B, depth, d, F, packed):
    """Batches of B * (depth + 1) rows at the edges of the few-row GEMM's row tiles (1 to 9
    row blocks, a second row tile, the last rows it takes and the first it does not), with
    few and many k units and k-slices, and partial row blocks of the activation layout."""
    w = small_bf16(d=d, F=F, B=B, S=40, tree="chain", depth=depth, V=5008 if packed else 5004)
    run = hz.run_tree(w, packed=packed)
    _check_tree(run, tol=2e-2)


@pytest.mark.parametrize("B, depth, F, V", [(17, 31, 13376, 26640), (9, 31, 576, 66000)])
def test_tree_wide_tiles(B, depth, F, V):
    """Packed gate/up and LM-head products whose rows fit 288-row tiles better than 128-row
    ones (544 rows: two tiles, the second partial; 288 rows: one), with a partial last
    column tile."""
    w = small_bf16(F=F, B=B, S=40, tree="chain", depth=depth, V=V, L=1)
    run = hz.run_tree(w, packed=True)
    _check_tree(run, tol=2e-2)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("B, depth, d, F", [
    (5, 59, 1024, 4096), (9, 32, 256, 13376), (12, 31, 512, 8192), (12, 31, 2048, 4096),
    (17, 31, 512, 8192)])
def test_tree_gate_up_tilings(B, depth, d, F, packed):
    """Gate/up beyond the few-row GEMM, 297 to 544 rows, at sizes whose least estimated time
    belongs to each of its tilings (288 x 256 tiles: the test above), one of them with
    k-slices; partial last row and column tiles."""
    w = small_bf16(d=d, F=F, B=B, S=40, tree="chain", depth=depth, V=2000, L=1)
    _check_tree(hz.run_tree(w, packed=packed), tol=2e-2)


@pytest.mark.parametrize("B, H, Hkv, S", [
    (1, 8, 8, 400), (1, 32, 8, 250), (2, 16, 8, 1520), (3, 8, 8, 3050), (3, 8, 8, 1100),
    (16, 8, 8, 300), (17, 8, 8, 600)])
def test_tree_key_splits(B, H, Hkv, S):
    """Attention over prefixes on either side of the rule that splits their keys: a few
    sessions in splits of 2 chunks or of 4, short prefixes that stay whole, and batches that
    leave no split or do not divide the CUs."""
    w = small_bf16(B=B, H=H, Hkv=Hkv, hd=128, S=S, ragged=False, V=1000, L=1)
    _check_tree(hz.run_tree(w), tol=2e-2)


@pytest.mark.parametrize("d, F", [(4096, 16384), (4096, 16448)])
def test_tree_wide_residual(d, F):
    """The row-major down projection of 297 rows at the widest weights that the few-row GEMM
    takes beyond 288 rows and at the narrowest that it leaves to the larger tiles."""
    w = small_bf16(d=d, F=F, B=9, S=40, tree="chain", depth=32, V=1000, L=1)
    _check_tree(hz.run_tree(w), tol=2e-2)


@pytest.mark.parametrize("B, depth, kw", [
    (1, 0, dict()), (2, 7, dict(d=64, F=64, H=1, Hkv=1, V=100)), (1, 16, dict(d=1024, F=2048)),
    (3, 20, dict(hd=128, H=2, Hkv=1, S=600)), (3, 48, dict(hd=128, H=4, Hkv=4, S=255, V=20004)),
    (5, 59, dict(S=30)), (2, 11, dict(d=8256, F=128, V=1000))])
def test_tree_fp32_shapes(B, depth, kw):
    """The fp32 model away from its one configuration: 1 to 300 rows (one to three row tiles
    of the GEMM), widths with one k unit and many, prefixes over several blocks of slots, a
    width beyond the fused residual norm, a vocabulary whose rows are split."""
    w = small_bf16(**dict(dict(dtype="f32", B=B, tree="chain", depth=depth, S=137, V=3004), **kw))
    _check_tree(hz.run_tree(w), tol=1e-4)


def test_pack_weight_layout_matches_its_definition():
    """acespec_pack_weight against the layout written out on the host: 16-byte unit
    u = (nb * cols/32 + kt) * 64 + l holds row nb*16 + l%16, columns kt*32 + (l/16)*8 .. +8,
    widened to fp16."""
    from paper_2609_02514_amd.acespec import Verifier, acespec_pack_weight
    rows, cols = 48, 96
    g = torch.Generator().manual_seed(7)
    src = (torch.randn(rows, cols, generator=g) * 0.05).to(torch.bfloat16)
    dst = torch.empty(rows * cols, dtype=torch.float16, device="cuda")
    srcd = src.cuda()
    acespec_pack_weight(srcd.data_ptr(), dst.data_ptr(), rows, cols, Verifier._stream())
    torch.cuda.synchronize()
    got = dst.cpu().numpy().reshape(rows // 16, cols // 32, 64, 8)
    ref = np.empty_like(got)
    s16 = src.to(torch.float16).numpy()
    for nb in range(rows // 16):
        for kt in range(cols // 32):
            for l in range(64):
                r, c = nb * 16 + l % 16, kt * 32 + (l // 16) * 8
                ref[nb, kt, l] = s16[r, c:c + 8]
    assert np.array_equal(got.view(np.uint16), ref.view(np.uint16))


def test_tree_empty_tree_and_long_ragged_prefix():
    """N = 0 (root only: bonus and top-k only) and prefixes that end mid-chunk."""
    w = small_bf16(tree="chain", depth=0, B=5, S=1000, ragged=True)
    run = hz.run_tree(w)
    _check_tree(run, tol=2e-2)
    assert run.outs["path_len"].tolist() == [0] * 5


@pytest.mark.timeout(900)
@pytest.mark.parametrize("seed", hz.parity_seeds(synth.get("1b-bf16"), 4))
def test_tree_1b_full_size(seed):
    """1B-class workload at full size, all 16 sessions through the oracle's forward."""
    w = synth.get("1b-bf16")
    # even seeds with packed weights (the benchmark's layout), odd ones row-major
    packed = (seed - w.seed_base) // 100 % 2 == 0
    run = hz.run_tree(w, seed=seed, packed=packed)
    _check_tree(run, tol=2e-2)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("seed", hz.parity_seeds(synth.get("8b-bf16"), 3))
def test_tree_8b_full_size(seed):
    """8B-class workload at full size: the oracle's forward on 4 sessions spread over the
    batch, decisions on all 64 sessions' 1088 rows."""
    w = synth.get("8b-bf16")
    i = (seed - w.seed_base) // 100
    run = hz.run_tree(w, seed=seed, sessions=[5 + i, 21 + i, 37 + i, 63 - i],
                      packed=i % 2 == 0)
    _check_tree(run, tol=2e-2)


@pytest.mark.timeout(900)
def test_tree_8b_geometric_tree():
    """A paper-shaped tree: main chain of 8 with 24 alternatives allocated by the geometric
    decay of Section IV (32 drafted nodes per session)."""
    w = synth.get("8b-geometric")
    run = hz.run_tree(w, sessions=[0, 23])
    _check_tree(run, tol=2e-2)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("seed", hz.parity_seeds(synth.get("8b-long-wide"), 3))
def test_tree_8b_long_wide(seed):
    """Long-context wide-tree workload at full size (16k-token prefixes, 64-node trees):
    the first seed runs the oracle's forward on all 8 sessions, the others on two."""
    w = synth.get("8b-long-wide")
    i = (seed - w.seed_base) // 100
    sessions = list(range(8)) if i == 0 else [2 * i, 7 - i]
    run = hz.run_tree(w, seed=seed, sessions=sessions, packed=i % 2 == 0)
    _check_tree(run, tol=2e-2)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("name", ["32b-bf16", "70b-bf16"])
def test_tree_paper_scale_widths(name):
    """The paper's cloud-target shapes (Qwen-32B / LLaMA-70B classes: d 5120 / 8192, G 5 / 8,
    vocab 152064 / 128256) at their full widths and batch, two layers deep: every kernel
    runs the launch configuration of the full-depth model (depth changes only the layer
    loop), and the float64 oracle stays within seconds per session."""
    w = synth.get(name).scaled(L=2)
    run = hz.run_tree(w, sessions=[11, 50], packed=name == "70b-bf16")
    _check_tree(run, tol=2e-2)


@pytest.mark.timeout(900)
def test_tree_70b_widths_64_node_tree():
    """The 70B-class widths (8 query heads per kv head) under the long-context workload's
    64-node tree: 520 query rows per kv head, more than one attention workgroup holds."""
    w = synth.get("70b-bf16").scaled(L=2, B=4, S=1024, tree="chain_sib", depth=8, sib=7,
                                     top_k=64, T=1.0, q_T=1.0, name="70b-wide")
    run = hz.run_tree(w, sessions=[1, 3], packed=True)
    _check_tree(run, tol=2e-2)


# ---------------------------------------------------------------------------------------
# LM-head tail
# ---------------------------------------------------------------------------------------


def _run_tail(w, W=None, rows_check=None, tol=1e-4, final_norm=False, seed=None,
              packed=False):
    """LM-head tail through the C ABI: logits of rows_check (default all) against the
    oracle's float64 LM head; decisions of EVERY row against the oracle's verify stage on
    the GPU's logits; the chain walk from the GPU's accept bits.  packed: the LM head in
    the packed layout (acespec_pack_weight), the oracle on the row-major matrix."""
    from paper_2609_02514_amd.acespec import Verifier
    dev = "cuda"
    seed = w.seed_base if seed is None else seed
    W = W or synth.make_weights(w, dev, seed)
    batch = synth.make_batch(w, dev, seed, weights=W)
    R = w.rows
    q_h, u_h, d_h = hz.host(batch.q), hz.host(batch.u), hz.host(batch.draft_tokens)
    v = Verifier.for_workload(w)
    outs = v.alloc_outputs(R, R // w.chain_len, w.chain_len, w.top_k, w.V, dev, True)
    hz.log(f"verify_tail R={R} V={w.V} seed={seed} packed={packed}")
    lm = v.pack_weights(W).lm_head if packed else W.lm_head
    v.verify_tail(lm, W.final_norm if final_norm else None, batch.hidden,
                  batch.draft_tokens, batch.q, batch.u, w.chain_len, w.T, w.top_p, w.top_k, outs,
                  packed=packed)
    torch.cuda.synchronize()
    del lm
    g = {k: (hz.host(t) if t is not None else None) for k, t in outs.items()}
    v.close()
    rows = list(range(R)) if rows_check is None else rows_check
    z_ref = om.lm_head_tail(W, batch.hidden[rows], final_norm=final_norm, eps=w.rms_eps)
    zg = g["logits_out"].numpy()
    err = hz.logits_rel_err(zg[rows].astype(np.float64), z_ref)
    hz.log(f"tail logits max rel err {err.max():.3e} over {len(rows)} rows")
    assert err.max() <= tol
    gn = {k: (t.numpy() if t is not None else None) for k, t in g.items()}
    rep = hz.check_rows(hz.tail_jobs(zg, q_h.numpy(), d_h.numpy(), u_h.numpy(), range(R),
                                     z_row_of=lambda r: r), gn, w.T, w.top_p, w.top_k)
    hz.log(f"tail decisions (all {R} rows): {rep}")
    info = hz.check_rows(hz.tail_jobs(z_ref, q_h.numpy(), d_h.numpy(), u_h.numpy(), rows),
                         gn, w.T, w.top_p, w.top_k)
    hz.log(f"informational, on the oracle's own logits ({len(rows)} rows): {info}")
    assert rep.ok(), str(rep)
    # chain walk from the GPU's own accept bits
    pl, nx = ov.walk_tail(g["accept"].numpy(), g["resample_token"].numpy(), w.chain_len)
    assert g["path_len"].tolist() == pl.tolist()
    assert g["next_token"].tolist() == nx.tolist()
    assert g["status"].tolist() == [0] * (R // w.chain_len)
    return g


def test_tail_small():
    w = synth.get("8b-lmhead-tail").scaled(name="tail-small", d=256, V=5004, rows=96,
                                          chain_len=8, top_k=16)
    _run_tail(w)


def test_tail_small_packed_lm_head():
    """The LM head in the packed layout (a vocabulary that is a multiple of 16), with a
    final norm: the same decisions as row-major against the oracle."""
    w = synth.get("8b-lmhead-tail").scaled(name="tail-packed", d=256, V=5008, rows=96,
                                          chain_len=8, top_k=16)
    W = synth.make_weights(w, "cuda")
    gain = 1.0 + synth.normal((w.d,), 0.1, torch.float32, "cuda", w.seed_base, 0, 2)
    W = dataclasses.replace(W, final_norm=gain.to(torch.bfloat16))
    _run_tail(w, W=W, tol=2e-3, final_norm=True, packed=True)


def test_tail_with_final_norm():
    """A non-NULL final_norm: the tail rows are RMS-normalised with the gain (rounded to
    fp16 for the LM head) before the product; the oracle normalises in float64."""
    w = synth.get("8b-lmhead-tail").scaled(name="tail-norm", d=256, V=5004, rows=64,
                                          chain_len=8, top_k=16)
    W = synth.make_weights(w, "cuda")
    gain = 1.0 + synth.normal((w.d,), 0.1, torch.float32, "cuda", w.seed_base, 0, 2)
    W = dataclasses.replace(W, final_norm=gain.to(torch.bfloat16))
    _run_tail(w, W=W, tol=2e-3, final_norm=True)


def test_tail_fp32_model_with_final_norm():
    """The fp32 model's tail (reference-precision kernels) with a final RMSNorm gain."""
    w = synth.get("8b-lmhead-tail").scaled(name="tail-f32", dtype="f32", d=192, V=3000,
                                          rows=48, chain_len=6, top_k=24)
    W = synth.make_weights(w, "cuda")
    gain = 1.0 + synth.normal((w.d,), 0.1, torch.float32, "cuda", w.seed_base, 0, 2)
    W = dataclasses.replace(W, final_norm=gain)
    _run_tail(w, W=W, tol=1e-4, final_norm=True)


@pytest.mark.parametrize("packed", [False, True])
def test_tail_exact_logit_ties(packed):
    """Duplicated LM-head rows give exactly equal logits (in either layout: every output
    column sums its products in the same order): ties must be broken by token id in the
    nucleus, the top-k payload and the inverse CDFs."""
    w = synth.get("8b-lmhead-tail").scaled(name="tail-ties", d=128, V=4096, rows=64,
                                          chain_len=4, top_k=32, T=1.0, top_p=0.5)
    W = synth.make_weights(w, "cuda")
    W.lm_head = W.lm_head[torch.arange(w.V, device="cuda") // 8].contiguous()
    _run_tail(w, W=W, packed=packed)


@pytest.mark.parametrize("rows, V, kind", [
    (1, 16384, "plain"), (32, 20000, "plain"), (128, 16640, "plain"), (129, 16384, "plain"),
    (40, 50004, "plain"), (512, 48000, "plain"), (513, 48000, "plain"),
    (32, 20000, "ties8"), (32, 20000, "ties24"), (32, 20000, "flat"), (32, 20000, "cold")])
def test_tail_split_rows(rows, V, kind):
    """Few rows of a large vocabulary are verified by several workgroups a row: at the edges
    of that rule, with ids tied at the thresholds (few: their ranks come from a list; many:
    the row is done whole), a nearly uniform target (the list overflows) and a near-greedy target
    (all but a few ids without mass)."""
    w = synth.get("8b-lmhead-tail").scaled(name="tail-split", d=128, V=V, rows=rows, chain_len=1,
                                          top_k=40, T={"cold": 0.03, "flat": 40.0}.get(kind, 0.8),
                                          top_p=1.0 if kind == "full" else 0.6)
    W = synth.make_weights(w, "cuda")
    if kind.startswith("ties"):
        n = int(kind[4:])
        W.lm_head = W.lm_head[torch.arange(w.V, device="cuda") // n].contiguous()
    _run_tail(w, W=W)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("rows, V, d, noalloc", [
    (1, 64, 64, False), (48, 4112, 512, False), (49, 4112, 512, True), (80, 50272, 256, False),
    (81, 50272, 256, False), (96, 4112, 4096, False), (96, 16400, 512, True),
    (129, 16400, 512, False), (160, 32016, 1024, True), (289, 8208, 2048, False),
    (272, 48016, 512, False), (288, 66000, 1024, False), (300, 32016, 256, False),
    (513, 16400, 1024, False), (577, 32016, 512, False)])
def test_lm_head_row_counts(rows, V, d, noalloc, packed):
    """The LM head's tilings, as its rows and vocabulary pick them: whole and sliced tiles of
    each size with a partial last row and column tile.  Logits against float64: a product of
    exact 16-bit inputs, d terms summed in fp32 in any order, each of magnitude 0.05 (d terms:
    their rounding errors, about 2^-24 of the running sum each, stay below d 2^-24 0.05 d^0.5;
    held to that).  The row maxima, which come from the tiles: the masses of the payload add up
    to one and the first id is the largest logit."""
    from paper_2609_02514_amd import acespec as A
    g = torch.Generator(device="cuda").manual_seed(rows + V)
    dt = torch.bfloat16
    hidden = torch.randn(rows, d, generator=g, device="cuda").to(dt)
    lm = (torch.randn(V, d, generator=g, device="cuda") * 0.05).to(dt)
    q = torch.full((rows, V), 1.0 / V, device="cuda")
    u = torch.full((rows, 3), 0.5, device="cuda")
    draft = torch.zeros(rows, dtype=torch.int32, device="cuda")
    outs = A.Verifier.alloc_outputs(rows, rows, 1, 4, V, "cuda", True)
    w, stream = lm, torch.cuda.current_stream().cuda_stream
    if packed:
        w = torch.empty(lm.numel(), dtype=torch.float16, device="cuda")
        A.acespec_pack_weight(lm.data_ptr(), w.data_ptr(), V, d, stream)
    hz.log(f"lm head R={rows} V={V} d={d} packed={packed} noalloc={noalloc}")
    if noalloc:
        A.acespec_verify_tail_noalloc(
            A.ModelDesc(0, d, 0, 1, 0, 0, V, 1e4, 1e-5, A.ACESPEC_BF16), w.data_ptr(),
            A.ACESPEC_LAYOUT_PACKED if packed else A.ACESPEC_LAYOUT_ROWS, None, hidden.data_ptr(),
            draft.data_ptr(), q.data_ptr(), u.data_ptr(), rows, 1, A.Params(1.0, 0.9, 4),
            A.Verifier.outputs_struct(outs), stream)
    else:
        v = A.Verifier(0, d, 0, 1, 0, 0, V, "bf16", rows, 0)
        v.verify_tail(w, None, hidden, draft, q, u, 1, 1.0, 0.9, 4, outs, packed=packed)
        torch.cuda.synchronize()
        v.close()
    torch.cuda.synchronize()
    assert (outs["status"] == 0).all()
    z = outs["logits_out"]
    want = hidden.double() @ lm.double().t()
    assert (z - want).abs().max() < d ** 1.5 * 2.0 ** -24 * 0.05
    assert torch.equal(z.gather(1, outs["topk_ids"][:, :1].long())[:, 0], z.max(1).values)
    assert ((outs["topk_probs"].sum(1) - 1).abs() < 1e-5).all()


def test_tail_fp32_activations_past_4_gib():
    """The fp32 model's hidden states beyond 2^32 bytes (262344 rows of width 4096), through
    the allocation-free entry point.  Bound of the logits: 4096 products of unit normals and
    weights of 0.02, summed in fp32 in any order: below 4096 * 2^-24 of the sum of magnitudes
    (52), 1.3e-2; about 1e-5 as the errors mostly cancel.  Held to 2e-4."""
    from paper_2609_02514_amd import acespec as A
    R, d, V, k = 262144 + 200, 4096, 64, 4
    g = torch.Generator(device="cuda").manual_seed(3)
    hidden = torch.randn(R, d, generator=g, device="cuda")
    lm = torch.randn(V, d, generator=g, device="cuda") * 0.02
    q = torch.full((R, V), 1.0 / V, device="cuda")
    u = torch.full((R, 3), 0.5, device="cuda")
    draft = torch.zeros(R, dtype=torch.int32, device="cuda")
    outs = A.Verifier.alloc_outputs(R, R, 1, k, V, "cuda", True)
    hz.log(f"noalloc tail fp32 R={R} d={d} V={V}")
    A.acespec_verify_tail_noalloc(
        A.ModelDesc(0, d, 0, 1, 0, 0, V, 1e4, 1e-5, A.ACESPEC_F32), lm.data_ptr(),
        A.ACESPEC_LAYOUT_ROWS, None, hidden.data_ptr(), draft.data_ptr(), q.data_ptr(),
        u.data_ptr(), R, 1, A.Params(0.8, 0.9, k), A.Verifier.outputs_struct(outs),
        torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert (outs["status"] == 0).all()
    for r0 in (0, 131072 - 100, R - 400):
        want = hidden[r0:r0 + 400].double() @ lm.double().t()
        assert (outs["logits_out"][r0:r0 + 400].double() - want).abs().max() < 2e-4, r0


@pytest.mark.parametrize("rows, V, kind", [
    (32, 20000, "plain"), (33, 20000, "plain"), (128, 24000, "plain"), (129, 24000, "plain"),
    (300, 96000, "plain"), (384, 48000, "full"), (385, 48000, "full"), (40, 7936, "plain"),
    (40, 8192, "plain"), (40, 7936, "ties8"), (40, 512, "flat")])
def test_tail_row_rules(rows, V, kind):
    """As above, at the edges of the rule by which rows are split (their number by the length
    of a row, where there are many by top_p), at two and three chunks a row, and where the last
    pass changes its form (8192 ids)."""
    test_tail_split_rows(rows, V, kind)


def _bin_edge(M, T, b):
    """The lowest float32 below M whose bin of the split passes (25 to the unit of the base-2
    exponent) is less than b bins below M's; its lower neighbour is in the next bin down."""
    c = np.float32(1.4426950408889634 / T)
    key = lambda z: int(np.float32(z).view(np.int32)) if z >= 0 else \
        -(int(np.float32(z).view(np.int32)) & 0x7FFFFFFF)
    val = lambda k: np.int32(k).view(np.float32) if k >= 0 else -np.int32(-k).view(np.float32)
    lo, hi = key(M - b * T), key(M)          # (lo: outside, hi: inside)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if (np.float32(val(mid) - M) * c) * np.float32(-25.0) < b:
            hi = mid
        else:
            lo = mid
    return key, val, hi


def _adjacent_bin_rows(T, V, n_up, n_down, seed):
    """Rows of logits whose order around an edge between two bins is decided by single ulps:
    the maximum, n_up ids from the edge upwards, n_down right below it, one id at the far end
    of either bin, the others without mass.  Maxima of all sizes, edges at and around zero
    among them (where floats are densest)."""
    rng = np.random.default_rng(seed)
    b, rows = 3, []
    for M in [10.0, 0.5, 1.0, 3.0, 40.0, -2.0, -0.3, -25.0, 0.0665, 0.07, 0.06, 0.0662] + \
            list(rng.uniform(-20, 20, 6)) + list(rng.uniform(0.02, 0.12, 6)):
        M = np.float32(M)
        key, val, e = _bin_edge(M, T, b)
        up_end, down_end = _bin_edge(M, T, b - 1)[2] - 1, _bin_edge(M, T, b + 1)[2]
        special = [val(up_end)] + [val(e + j) for j in range(n_up)] + \
            [val(e - 1 - j) for j in range(n_down)] + [val(down_end)]
        z = (M - np.float32(30.0) - rng.random(V).astype(np.float32)).astype(np.float32)
        at = rng.choice(V, len(special) + 1, replace=False)
        z[at] = [M] + special
        rows.append(z)
    return np.stack(rows)


def _run_given_logits(z, reps, q, draft, u, T, top_p, top_k):
    """The tail over exactly these logits (fp32 model, LM head z^T, one-hot hidden states),
    every row reps times over."""
    from paper_2609_02514_amd.acespec import Verifier
    n, V = z.shape
    R, d = n * reps, 64
    lm = torch.zeros(V, d)
    lm[:, :n] = torch.from_numpy(z).t()
    hidden = torch.eye(n, d).repeat(reps, 1).cuda()
    v = Verifier(0, d, 0, 1, 0, 0, V, "f32", R, 0)
    outs = v.alloc_outputs(R, R, 1, top_k, V, "cuda", True)
    dev = lambda t: torch.from_numpy(t).repeat(reps, *([1] * (t.ndim - 1))).cuda()
    hz.log(f"given logits: R={R} V={V} T={T} top_p={top_p:.6f} top_k={top_k}")
    v.verify_tail(lm.cuda(), None, hidden, dev(draft), dev(q), dev(u), 1, T, top_p, top_k, outs)
    torch.cuda.synchronize()
    v.close()
    return {k: t.cpu().numpy()[:n] for k, t in outs.items()}


@pytest.mark.parametrize("lower", ["top_k", "top_p"])
def test_tail_split_rows_thresholds_in_adjacent_bins(lower):
    """One threshold on the highest id of a bin, the other in the next bin up, a few ulps
    away: the ids of the upper bin are not part of the lower threshold's search.  Split rows
    against the ids in sorted order, and against the whole-row kernel (more rows of the same
    logits than are split), bit for bit."""
    T, V, n_up, n_down = 0.8, 24000, 8, 6
    z = _adjacent_bin_rows(T, V, n_up, n_down, 11)
    n = len(z)
    order = np.stack([np.lexsort((np.arange(V), -r)) for r in z])
    zs = np.take_along_axis(z.astype(np.float64), order, 1)
    p = np.exp((zs - zs[:, :1]) / T)
    cum = (p.cumsum(1) / p.sum(1, keepdims=True)).mean(0)   # (the same rows to 1e-4)
    first_down = 2 + n_up            # rank of the highest id of the lower bin
    if lower == "top_k":
        top_k, cross = first_down + 1, 3
    else:
        top_k, cross = 4, first_down
    top_p = float(0.5 * (cum[cross - 1] + cum[cross]))
    rng = np.random.default_rng(5)
    q = rng.random((n, V)).astype(np.float32)
    q /= q.sum(1, keepdims=True)
    draft = order[np.arange(n), rng.integers(0, 12, n)].astype(np.int32)
    u = rng.uniform(0.01, 0.99, (n, 3)).astype(np.float32)
    split = _run_given_logits(z, 1, q, draft, u, T, top_p, top_k)
    whole = _run_given_logits(z, 6, q, draft, u, T, top_p, top_k)
    assert np.array_equal(split["logits_out"], z) and (split["status"] == 0).all()
    for g in (whole, split):
        assert np.array_equal(g["topk_ids"], order[:, :top_k])
        # ids up to the crossing one carry mass, no others
        assert ((g["topk_probs"] > 0) == (np.arange(top_k) <= cross)).all()
    for k in split:
        assert np.array_equal(split[k], whole[k]), k


@pytest.mark.parametrize("T,top_p,top_k", [
    (1.0, 1.0, 256),    # whole vocabulary in the nucleus, the largest payload
    (0.05, 0.9, 1),     # near-greedy target, a one-token payload
    (4.0, 0.3, 8),      # flat target, a nucleus of a small mass fraction
    (0.8, 0.999, 200),  # nucleus boundary deep in the tail
])
def test_tail_parameter_extremes(T, top_p, top_k):
    """Section III-B's sampling parameters at the ends of their ranges (temperature,
    nucleus mass, payload size), on the same decisions as the other tail tests."""
    w = synth.get("8b-lmhead-tail").scaled(name="tail-extremes", d=256, V=5004, rows=64,
                                          chain_len=4, top_k=top_k, T=T, top_p=top_p)
    _run_tail(w)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("seed", hz.parity_seeds(synth.get("8b-lmhead-tail"), 3))
def test_tail_8b_full_size(seed):
    """The LM-head tail at full size (4096 rows, vocab 128256): decisions on all rows,
    the float64 LM head on 512 sampled rows; even seeds with the packed LM head (the
    benchmark's layout), odd ones row-major."""
    w = synth.get("8b-lmhead-tail")
    rng = np.random.default_rng(seed)
    rows = sorted(rng.choice(w.rows, 512, replace=False).tolist())
    packed = (seed - w.seed_base) // 100 % 2 == 0
    g = _run_tail(w, rows_check=rows, tol=1e-4, seed=seed, packed=packed)
    rate = float(g["accept"].float().mean())
    hz.log(f"tail acceptance rate {rate:.3f}")
    assert 0.3 < rate < 0.95


# ---------------------------------------------------------------------------------------
# ABI behaviour on the device
# ---------------------------------------------------------------------------------------


def test_bad_trees_flag_only_their_session():
    from paper_2609_02514_amd.acespec import Verifier
    w = small_bf16(B=4, ragged=False)
    W = synth.make_weights(w, "cuda")
    batch = synth.make_batch(w, "cuda")
    par = batch.parents.clone()
    tok = batch.tokens.clone()
    par[1, 5] = 7          # forward reference
    tok[2, 3] = w.V + 3    # token outside the vocabulary
    plen = batch.prefix_len.clone()
    plen[3] = batch.cap    # prefix leaves no room for the tree
    v = Verifier.for_workload(w)
    B, n1 = tok.shape
    outs = v.alloc_outputs(B * n1, B, n1, w.top_k, w.V, "cuda", False)
    v.verify_tree(v.weights_struct(W), batch.kv_k, batch.kv_v, batch.cap, plen, tok, par,
                  batch.q, batch.u, w.T, w.top_p, w.top_k, outs)
    torch.cuda.synchronize()
    assert outs["status"].tolist() == [0, -5, -5, -5]
    v.close()


def test_argument_errors_are_synchronous():
    from paper_2609_02514_amd import acespec as A
    w = small_bf16(B=2)
    W = synth.make_weights(w, "cuda")
    batch = synth.make_batch(w, "cuda")
    v = A.Verifier.for_workload(w)
    B, n1 = batch.tokens.shape
    outs = v.alloc_outputs(B * n1, B, n1, w.top_k, w.V, "cuda", False)
    ws = v.weights_struct(W)
    for T, top_p, k, code in [(0.0, 0.9, 8, -1), (0.8, 0.0, 8, -1), (0.8, 1.5, 8, -1),
                              (0.8, 0.9, 0, -1), (0.8, 0.9, 300, -1)]:
        with pytest.raises(A.AcespecError) as e:
            v.verify_tree(ws, batch.kv_k, batch.kv_v, batch.cap, batch.prefix_len,
                          batch.tokens, batch.parents, batch.q, batch.u, T, top_p, k, outs)
        assert e.value.code == code
    with pytest.raises(A.AcespecError):   # more sessions than the context holds
        big = batch.tokens.repeat(3, 1)
        v.verify_tree(ws, batch.kv_k, batch.kv_v, batch.cap, batch.prefix_len, big,
                      batch.parents.repeat(3, 1), batch.q, batch.u, 0.8, 0.9, 8, outs)
    v.close()
    with pytest.raises(A.AcespecError) as e:
        A.Verifier(1, 256, 4, 4, 96, 512, 1000, "bf16", 2, 4)   # head_dim 96
    assert e.value.code == -2


def test_run_to_run_bitwise_determinism():
    from paper_2609_02514_amd.acespec import Verifier
    w = small_bf16(B=2)
    W = synth.make_weights(w, "cuda")
    batch = synth.make_batch(w, "cuda")
    v = Verifier.for_workload(w)
    B, n1 = batch.tokens.shape
    ws = v.weights_struct(W)
    res = []
    for _ in range(2):
        outs = v.alloc_outputs(B * n1, B, n1, w.top_k, w.V, "cuda", True)
        v.verify_tree(ws, batch.kv_k, batch.kv_v, batch.cap, batch.prefix_len, batch.tokens,
                      batch.parents, batch.q, batch.u, w.T, w.top_p, w.top_k, outs)
        torch.cuda.synchronize()
        res.append({k: t.clone() for k, t in outs.items() if t is not None})
    for k in res[0]:
        assert torch.equal(res[0][k], res[1][k]), k
    v.close()


def test_timing_selection():
    """acespec_timing_only restricts the recorded kernels to one kind; unknown kinds are
    rejected synchronously; NULL restores every kind."""
    from paper_2609_02514_amd import acespec as A
    w = small_bf16(B=2)
    W = synth.make_weights(w, "cuda")
    batch = synth.make_batch(w, "cuda")
    v = A.Verifier.for_workload(w)
    B, n1 = batch.tokens.shape
    ws = v.weights_struct(W)
    outs = v.alloc_outputs(B * n1, B, n1, w.top_k, w.V, "cuda", False)

    def step():
        v.verify_tree(ws, batch.kv_k, batch.kv_v, batch.cap, batch.prefix_len, batch.tokens,
                      batch.parents, batch.q, batch.u, w.T, w.top_p, w.top_k, outs)

    A.acespec_timing_enable(v.ctx, True)
    A.acespec_timing_only(v.ctx, "gemm_gate_up")
    A.acespec_timing_read(v.ctx)
    step()
    got = A.acespec_timing_read(v.ctx)
    assert list(got) == ["gemm_gate_up"] and got["gemm_gate_up"][1] == w.L
    with pytest.raises(A.AcespecError) as e:
        A.acespec_timing_only(v.ctx, "no_such_kernel")
    assert e.value.code == -1
    A.acespec_timing_only(v.ctx, None)
    step()
    got = A.acespec_timing_read(v.ctx)
    assert {"gemm_gate_up", "tree_attention", "vocab_verify", "path_walk"} <= set(got)
    A.acespec_timing_enable(v.ctx, False)
    v.close()
