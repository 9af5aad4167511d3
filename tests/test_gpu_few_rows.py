"""Products on few rows (ring tiles, K split over workgroups): the forward pass against the oracle at
the row counts where the tile or the split changes (1, 64 and 65 rows; residual projections: 32 x 32
tiles up to 128 rows, then MLP down split three ways up to 512 where its K is 2048 or more, two ways up
to 1024, not split from 1025 on; 2048 and 2049), at K-tiles that are ragged (d_mlp and adapter ranks that
are no multiple of 64), and the loop's listed rows against the full path.

Bar: as for every forward pass, max |dlogit| <= 5e-2 in bf16 (measured here up to 1.3e-2)."""
import numpy as np
import pytest

import workloads
from oracle import forward as oforward, params as oparams
from tests.gpu_util import dev_i32, say, torch_or_skip

from paper_2609_04010_amd import _lib as dd

pytestmark = pytest.mark.gpu

TOL = 5e-2

CASES = [
    # overrides of the GPT-2-small shape, B, L
    (dict(n_layers=2, vocab=300), 1, 1),
    (dict(n_layers=2, vocab=300), 1, 64),
    (dict(n_layers=2, vocab=300), 5, 13),
    (dict(n_layers=1, vocab=300), 2, 256),
    (dict(n_layers=1, vocab=300), 3, 171),
    (dict(n_layers=1, vocab=300), 8, 256),
    (dict(n_layers=1, vocab=300), 3, 683),
    # one ragged K-tile (40, 8 and 56 of 64), not split
    (dict(n_layers=1, vocab=300, d_mlp=1000), 1, 70),
    (dict(n_layers=1, vocab=300, d_mlp=520), 3, 200),
    (dict(n_layers=1, vocab=300, d_mlp=120), 5, 500),
    (dict(n_layers=2, vocab=300, lora_rank=8, lora_alpha=16.0), 1, 90),
    (dict(n_layers=1, vocab=300, lora_rank=72, lora_alpha=144.0), 3, 250),
    # other widths, K of one to eight K-tiles
    (dict(n_layers=2, vocab=300, d_model=64, n_heads=1, d_mlp=256), 2, 40),
    (dict(n_layers=2, vocab=300, d_model=256, n_heads=4, d_mlp=256), 2, 100),
    (dict(n_layers=2, vocab=300, d_model=512, n_heads=8, d_mlp=2048, norm="rms"), 2, 150),
    # the widths the four-features-per-lane normalisation takes besides 768 and 1024
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4, d_mlp=256, norm="rms"), 1, 33),
    (dict(n_layers=1, vocab=300, d_model=1536, n_heads=24, d_mlp=256), 2, 70),
    # MLP down at 128, 129, 1024 and 1025 rows
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4), 1, 128),
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4), 3, 43),
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4), 2, 512),
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4), 5, 205),
    # a ragged K-tile (56 of 64; 24 adapter columns after it) in the last of three splits, then of two
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4, d_mlp=2104), 1, 150),
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4, d_mlp=2104), 2, 256),
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4, d_mlp=2104), 3, 171),
    (dict(n_layers=1, vocab=300, d_model=256, n_heads=4, d_mlp=3000, lora_rank=24, lora_alpha=48.0), 2, 200),
    # a residual projection on 128 x 192 tiles (attention output), ragged rows and columns
    (dict(n_layers=1, vocab=64, d_model=256, n_heads=4, d_mlp=1024), 53, 238),
    # 128 x 192 tiles with ragged rows, columns and K (MLP up)
    (dict(n_layers=1, vocab=300, lora_rank=8, lora_alpha=16.0), 7, 241),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"B{c[1]}-L{c[2]}-" + "-".join(f"{k}{v}" for k, v in c[0].items()))
def test_forward_on_few_rows_matches_oracle(case):
    torch = torch_or_skip()
    over, B, L = case
    say("few rows", case)
    cfg = workloads.model_cfg(2, max_len=L, **over)
    P = oparams.init_params(cfg, 41)
    blob = dd.pack_params(cfg, oparams.storage_tensors(cfg, P))
    buf = torch.zeros(blob.size, dtype=torch.uint8, device="cuda")
    dd.init_params(cfg, buf, host_blob=blob)
    z = workloads.masked_state(77, B, L, cfg["vocab"], 0.5)
    ld = int(dd.logits_ld(cfg["vocab"]))
    logits = torch.zeros((B * L, ld), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((dd.workspace_bytes(cfg, B, L),), 0xFF, dtype=torch.uint8, device="cuda")   # NaN bits
    dd.workspace_reset(ws)
    zd = dev_i32(torch, z.reshape(-1))
    dd.denoise_forward(cfg, buf, zd, B, L, 0.5, logits, ld, ws)
    first = logits.clone()
    dd.denoise_forward(cfg, buf, zd, B, L, 0.5, logits, ld, ws)
    assert torch.equal(first, logits)          # sums in a fixed order
    got = first[:, :cfg["vocab"]].float().cpu().numpy().reshape(B, L, -1)
    assert dd.read_device_error(ws[:4].view(torch.int32)) == 0
    ref = oforward.forward(cfg, P, z, 0.5)
    err = float(np.abs(got - ref).max())
    say(f"max |dlogit| = {err:.3e}")
    assert err <= TOL


ATTN_CASES = [
    # B, L, pattern, block (12 heads): the key groups of the attention at the lines between 4, 2 and 1
    # groups, groups without a tile, ragged last tiles
    (1, 65, None, 0), (1, 130, "causal", 0), (1, 200, "draft_train", 4),
    (5, 256, None, 0), (6, 256, "block_causal", 48), (2, 641, None, 0), (2, 641, "causal", 0),
    (1, 2049, "causal", 0), (1, 2049, None, 0), (22, 129, None, 0), (22, 130, "draft_train", 13),
    # between one and two query blocks per CU on a long sequence: two groups under a pattern only
    (2, 2049, None, 0), (2, 2049, "causal", 0), (2, 2050, "draft_train", 41),
]


@pytest.mark.parametrize("case", ATTN_CASES, ids=lambda c: f"B{c[0]}-L{c[1]}-{c[2]}")
def test_attention_key_groups_match_oracle(case):
    """One layer whose attention weights are large enough (x 8) that its probabilities are not flat.
    Bar as above."""
    torch = torch_or_skip()
    B, L, pattern, block = case
    say("attention", case)
    cfg = workloads.model_cfg(2, n_layers=1, vocab=64, d_mlp=128, max_len=L)
    P = oparams.init_params(cfg, 44)
    P["l0.w_qkv"] = P["l0.w_qkv"].copy()
    P["l0.w_qkv"][:2 * cfg["d_model"]] *= 8.0      # exact in bf16
    blob = dd.pack_params(cfg, oparams.storage_tensors(cfg, P))
    buf = torch.zeros(blob.size, dtype=torch.uint8, device="cuda")
    dd.init_params(cfg, buf, host_blob=blob)
    z = workloads.masked_state(79, B, L, cfg["vocab"], 0.3)
    ld = int(dd.logits_ld(cfg["vocab"]))
    logits = torch.zeros((B * L, ld), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((dd.workspace_bytes(cfg, B, L),), 0xFF, dtype=torch.uint8, device="cuda")
    dd.workspace_reset(ws)
    vis, mask = None, None
    if pattern:
        host = dd.attn_mask_build(pattern, L, block)
        mask = dev_i32(torch, host.reshape(-1))
        j = np.arange(L)[None, :]
        vis = (j < host[0][:, None]) | ((j >= host[1][:, None]) & (j < host[2][:, None]))
    dd.denoise_forward_ex(cfg, buf, dev_i32(torch, z.reshape(-1)), B, L, 0.5, logits, ld, ws, attn_mask=mask)
    got = logits[:, :cfg["vocab"]].float().cpu().numpy().reshape(B, L, -1)
    assert dd.read_device_error(ws[:4].view(torch.int32)) == 0
    err = float(np.abs(got - oforward.forward(cfg, P, z, 0.5, vis)).max())
    say(f"max |dlogit| = {err:.3e}")
    assert err <= TOL


F32_CASES = [
    # d_model, heads (head dim 16 / 32 / 64 / 128), layers, B, L, pattern, block
    (64, 4, 2, 3, 1, None, 0),
    (64, 4, 2, 2, 33, "causal", 0),
    (64, 2, 2, 2, 130, None, 0),
    (128, 2, 2, 2, 31, "block_causal", 5),
    (256, 2, 2, 1, 160, "draft_train", 8),
    (256, 4, 1, 2, 257, None, 0),
    (768, 12, 1, 5, 120, None, 0),      # 600 rows: residual projections on 64 x 64 tiles, not split
    (256, 4, 1, 4, 120, None, 0),       # 480 rows: on 32 x 64 tiles with K over two pairs of wavefronts
]


@pytest.mark.parametrize("case", F32_CASES, ids=lambda c: f"d{c[0]}-h{c[1]}-B{c[3]}-L{c[4]}-{c[5]}")
def test_fp32_forward_matches_oracle(case):
    """The matrix-core fp32 GEMM and attention: every head dim, key and query tails, patterns.  Bar: the
    validation build's 1e-4; fp32 sums of these lengths leave about 1e-6."""
    torch = torch_or_skip()
    d, H, nl, B, L, pattern, block = case
    say("fp32", case)
    cfg = workloads.model_cfg(1, d_model=d, n_heads=H, n_layers=nl, d_mlp=4 * d - 8, vocab=77, max_len=L)
    P = oparams.init_params(cfg, 43)
    blob = dd.pack_params(cfg, oparams.storage_tensors(cfg, P))
    buf = torch.zeros(blob.size, dtype=torch.uint8, device="cuda")
    dd.init_params(cfg, buf, host_blob=blob)
    z = workloads.masked_state(78, B, L, cfg["vocab"], 0.5)
    ld = int(dd.logits_ld(cfg["vocab"]))
    logits = torch.zeros((B * L, ld), dtype=torch.float32, device="cuda")
    ws = torch.full((dd.workspace_bytes(cfg, B, L),), 0xFF, dtype=torch.uint8, device="cuda")
    dd.workspace_reset(ws)
    vis, mask = None, None
    if pattern:
        host = dd.attn_mask_build(pattern, L, block)
        mask = dev_i32(torch, host.reshape(-1))
        j = np.arange(L)[None, :]
        vis = (j < host[0][:, None]) | ((j >= host[1][:, None]) & (j < host[2][:, None]))
    dd.denoise_forward_ex(cfg, buf, dev_i32(torch, z.reshape(-1)), B, L, 0.5, logits, ld, ws, attn_mask=mask)
    got = logits[:, :cfg["vocab"]].double().cpu().numpy().reshape(B, L, -1)
    assert torch.all(logits[:, cfg["vocab"]:] == 0)
    assert dd.read_device_error(ws[:4].view(torch.int32)) == 0
    err = float(np.abs(got - oforward.forward(cfg, P, z, 0.5, vis)).max())
    say(f"max |dlogit| = {err:.3e}")
    assert err <= 1e-4


LISTED_CASES = [
    # overrides, B, L, T: the row counts on either side of the lines of the residual projections' split
    # (128, 512, 1024 rows), and above 2048, where the layer is launched for many and for few listed rows
    (dict(d_model=128, n_heads=2, vocab=12000), 1, 40, 3),
    (dict(d_model=128, n_heads=2, vocab=12000), 2, 64, 3),
    (dict(d_model=128, n_heads=2, vocab=12000), 3, 43, 3),
    (dict(d_model=128, n_heads=2, vocab=12000, d_mlp=128), 3, 50, 3),    # no room for a slab beside the MLP rows
    (dict(), 1, 150, 3),
    (dict(), 2, 256, 3),
    (dict(), 3, 200, 3),
    (dict(), 4, 275, 3),
    (dict(), 7, 300, 3),
    (dict(), 7, 300, 1),      # every row listed: the 256-row tiles
]


@pytest.mark.parametrize("case", LISTED_CASES, ids=lambda c: f"B{c[1]}-L{c[2]}-T{c[3]}-" + "-".join(f"{k}{v}" for k, v in c[0].items()))
def test_listed_rows_have_the_full_path_logits(case):
    """The loop's last layer runs on the listed rows alone; their logits are those of
    dd_denoise_forward on every row, bit for bit.  Compared where the vocabulary projection sums K in
    the same order on both sides: list index and token row both in the first tile of 256 rows."""
    torch = torch_or_skip()
    over, B, L, T = case
    say("listed rows", case)
    cfg = workloads.model_cfg(2, n_layers=2, max_len=L, **over)
    V, M = cfg["vocab"], B * L
    buf = torch.zeros(dd.param_bytes(cfg), dtype=torch.uint8, device="cuda")
    dd.init_params(cfg, buf, seed=45)
    al = 1.0 - np.arange(T + 1) / T
    z = torch.full((M,), V, dtype=torch.int32, device="cuda")
    trace = torch.zeros((T + 1, M), dtype=torch.int32, device="cuda")
    ws = torch.full((dd.loop_workspace_bytes(cfg, B, L),), 0xFF, dtype=torch.uint8, device="cuda")
    dd.workspace_reset(ws)
    dd.sample_loop(cfg, buf, B, L, T, al, z, ws, noise_seed=5, z_trace=trace)
    lay = dd.loop_workspace_layout(cfg, B, L)
    ld = lay["logits_ld"]
    count = int(ws[lay["count"]:lay["count"] + 4].view(torch.int32).item())
    rows = ws[lay["rows"]:lay["rows"] + 4 * count].view(torch.int32).long()
    got = ws[lay["logits"]:lay["logits"] + 2 * count * ld].view(torch.bfloat16).view(count, ld)[:, :V]
    full = torch.zeros((M, ld), dtype=torch.bfloat16, device="cuda")
    ws_f = torch.zeros(dd.workspace_bytes(cfg, B, L), dtype=torch.uint8, device="cuda")
    dd.denoise_forward(cfg, buf, trace[T - 1].clone(), B, L, al[1], full, ld, ws_f)
    first = rows[:256][rows[:256] < 256]
    say(f"{count} listed rows of {M}, {first.numel()} compared")
    assert count == int((trace[T - 1] == V).sum()) and first.numel() > 0
    assert torch.equal(got[:first.numel()], full[first][:, :V])
