"""Shared by CPU and GPU tests: properties the work units of a plan must have, whatever shape the
kernels give their work items.

`lora_plan_dump` returns the units decoded from the buffer the kernels read.  The slot/segment
indexing is right exactly when these units, taken together, say for every token what the
oracle's `token_map` says (which slot, which rank) and cover the work once:

* tile units: the tokens, slot and rank of the oracle's tiles, tile by tile (the tile/group
  partition under the plan's threshold is part of the library's contract);
* GEMV units: their tokens are the tokens of the oracle's groups; per token the shrink units cover
  rank rows [0, rank) exactly once (rows of the zero padding up to the next multiple of 8 at most
  once) and, per projection, the expand units cover columns [0, h_out) exactly once;
  the same holds for the units of a list call's batch, entry by entry, with the items and with the wide items;
* units of a short tile shrink: every (tile token, rank row) once, in units of at most 16 x 16, and they are marked as what a call works
  through exactly where it takes in no more than 225 MB that way;
* units of a shrink by panels: per number of projections that share it, every tile's tokens once per projection;
* row units of the fused linear path: every token of the batch exactly once.

The same holds for the lists with tiles that a plan holds besides its own (`lora_plan_dump_tiled`, threshold 8), which have no run tables.
"""
from __future__ import annotations

import numpy as np

import oracle
from paper_2411_17741_amd import binding as B


def check_plan_units(cache, plan, T, seg_offsets, seg_slot, seg_rank, projs, alpha_of_slot, bf16=True, tiled=False):
    """projs: [(h_in, h_out)]; alpha_of_slot: dict slot -> alpha; tiled: of the lists with tiles besides the plan's own.  Returns a dict of counts."""
    rc, info = B.lora_plan_info(plan)
    assert rc == B.LORA_OK
    if tiled:
        assert info.n_tiles == 0
        info.mfma_min_tokens = B.LORA_MFMA_MIN_TOKENS_MIXED
    tm_slot, tm_rank = (np.asarray(v, np.int64) for v in oracle.token_map(T, seg_offsets, seg_slot, seg_rank))
    want = oracle.index(T, seg_offsets, seg_slot, seg_rank, info.mfma_min_tokens)
    want_tile_toks = [want["tok_list"][o : o + n] for (o, n, *_r) in want["tiles"]]
    want_gemv = sorted(t for (o, n, *_r) in want["groups"] for t in want["tok_list"][o : o + n])
    gemv_pos = {t: i for i, t in enumerate(want_gemv)}
    counts = {}
    for p, (h_in, h_out) in enumerate(projs):
        rc, units, toks = (B.lora_plan_dump_tiled if tiled else B.lora_plan_dump)(cache, plan, p)
        assert rc == B.LORA_OK
        assert (units["tok_off"] >= 0).all() and (units["tok_off"] + units["n_tok"] <= len(toks)).all()
        assert ((toks >= 0) & (toks < T)).all()
        toks_of = lambda u: toks[u["tok_off"] : u["tok_off"] + u["n_tok"]]

        def same_entry(u):
            tk = toks_of(u)
            assert u["n_tok"] >= 1
            assert (tm_slot[tk] == u["slot"]).all() and (tm_rank[tk] == u["rank"]).all(), (u, tk)
            assert u["alpha"] == np.float32(alpha_of_slot[int(u["slot"])])

        # --- tiles: the oracle's, in order
        tiles = units[units["kind"] == B.LORA_UNIT_TILE]
        assert len(tiles) == len(want["tiles"]) and (len(tiles) > 0 if tiled else len(tiles) == info.n_tiles)
        for u, wt, (_, _, slot, rank, _, _) in zip(tiles, want_tile_toks, want["tiles"]):
            assert list(toks_of(u)) == wt and (u["slot"], u["rank"]) == (slot, rank)
            assert 1 <= u["n_tok"] <= B.LORA_TILE_TOKENS
            same_entry(u)

        # --- short tile shrink
        direct = units[units["kind"] == B.LORA_UNIT_DIRECT_SHRINK]
        if len(direct):
            cover = np.zeros((T, B.LORA_MAX_RANK), np.int8)
            for u in direct:
                same_entry(u)
                assert u["n_tok"] <= 16 and 0 <= u["lo"] < u["hi"] <= u["lo"] + 16 and u["hi"] <= u["rank"] and u["lo"] % 16 == 0
                assert len(set(toks_of(u))) == u["n_tok"]
                cover[toks_of(u), u["lo"] : u["hi"]] += 1
            in_tiles = np.asarray(sorted(t for tk in want_tile_toks for t in tk), np.int64)
            want_cover = np.zeros_like(cover)
            for t in in_tiles:
                want_cover[t, : tm_rank[t]] = 1
            assert (cover == want_cover).all()
            assert (direct["where"] == (len(direct) * 64 * h_in <= 225000000)).all()
        elif len(tiles) and bf16:  # none: more than a plan has room for
            n = sum(-(-len(tk) // 16) * -(-int(r) // 16) for tk, (_o, _n, _s, r, _t, _l) in zip(want_tile_toks, want["tiles"]))
            assert n > 2048 or n * 64 * min(i for i, _o in projs) > 225000000

        # --- shrink by panels: every tile token once per projection of a group of 1 to 4
        panels = units[units["kind"] == B.LORA_UNIT_PANEL_SHRINK]
        ways = units[units["kind"] == B.LORA_UNIT_SHRINK_WAY]
        assert list(ways["where"]) == ([1, 2, 3, 4] if len(tiles) else [])
        assert ((ways["lo"] == 0) == np.asarray([bool(len(direct)) and len(direct) * 64 * h_in * n <= 225000000 for n in ways["where"]])).all()
        assert (len(panels) > 0) == (len(tiles) > 0)  # (a plan has room for them whatever its batch)
        assert not (tiled and (ways["lo"] == 1).any())
        for gn in range(1, 5) if len(panels) else ():
            cover = np.zeros((gn, T), np.int32)
            for u in panels[panels["where"] == gn]:
                same_entry(u)
                assert u["n_tok"] <= 192 and 0 <= u["lo"] < u["hi"] <= gn
                cover[u["lo"] : u["hi"], toks_of(u)] += 1
            assert cover.sum() == gn * sum(len(tk) for tk in want_tile_toks) and (cover[:, [t for tk in want_tile_toks for t in tk]] == 1).all()

        # --- tile shrink: under every run table the pieces of a tile cover its input columns [0, h_in) once, in pieces
        # of whole 128-column stages; runs are walked in order, each at most a tail, whole tiles and a head; pieces that
        # are not whole tiles leave partial sums in slots of their own, and the reduce adds up exactly those
        pieces = units[units["kind"] == B.LORA_UNIT_TILE_SHRINK]
        sums = units[units["kind"] == B.LORA_UNIT_TILE_SUM]
        tile_of_off = {int(u["tok_off"]): i for i, u in enumerate(tiles)}
        for table in range(7):
            pc = pieces[(pieces["where"] >> 20) == table]
            sm = sums[(sums["where"] >> 20) == table]
            if len(tiles) == 0 or tiled or (table == 4 and T > B.LORA_STATIC_MAX_TOKENS):  # (no table for what the call refuses)
                assert len(pc) == 0 and len(sm) == 0
                continue
            runs = pc["where"] & 0xFFFFF
            assert (np.diff(runs) >= 0).all() and runs.max() < [512, 512 // 2, 512 // 3, 512 // 4, 128, 64, 32][table]
            cover = np.zeros((len(tiles), h_in), np.int8)
            slots_of_tile = [[] for _ in tiles]
            order = []
            for u in pc:
                i = tile_of_off[int(u["tok_off"])]
                assert (u["n_tok"], u["slot"], u["rank"]) == (tiles[i]["n_tok"], tiles[i]["slot"], tiles[i]["rank"])
                assert 0 <= u["lo"] < u["hi"] <= h_in and u["lo"] % 128 == 0 and (u["hi"] % 128 == 0 or u["hi"] == h_in)
                cover[i, u["lo"] : u["hi"]] += 1
                whole = u["lo"] == 0 and u["hi"] == h_in
                assert (u["alpha"] == -1) == whole
                if not whole:
                    assert u["hi"] - u["lo"] >= min(256, h_in // 2), u  # no slivers
                    slots_of_tile[i].append(int(u["alpha"]))
                order.append((i, int(u["lo"])))
            assert (cover == 1).all()
            assert order == sorted(order)  # the runs walk the tiles' columns in order
            all_slots = [s for l in slots_of_tile for s in l]
            assert len(set(all_slots)) == len(all_slots) and all(0 <= s < 2 * (int(runs.max()) + 1) for s in all_slots)
            for r in np.unique(runs):  # a run leaves at most two partial sums
                assert (pc[runs == r]["alpha"] >= 0).sum() <= 2
            got = [[] for _ in tiles]
            for u in sm:
                i = tile_of_off[int(u["tok_off"])]
                assert u["lo"] == len(got[i]) and u["hi"] == len(slots_of_tile[i])
                got[i].append(int(u["alpha"]))
            assert got == slots_of_tile

        # --- GEMV shrink: every (token, rank row) once; expand: every (token, output column) once.  The launch of this
        # projection alone, and every entry of a batch, with either kind of items
        def covers_once(gs, ge, max_rows, max_tok_s, max_tok_e):
            cover = np.zeros((len(want_gemv), B.LORA_MAX_RANK), np.int32)
            for u in gs:
                same_entry(u)
                assert 0 <= u["lo"] < u["hi"] <= (u["rank"] + 7) // 8 * 8 and u["hi"] - u["lo"] <= max_rows and u["n_tok"] <= max_tok_s
                idx = [gemv_pos[int(t)] for t in toks_of(u)]  # KeyError: a token that is not on the GEMV path
                assert len(set(idx)) == len(idx)
                cover[idx, u["lo"] : u["hi"]] += 1
            for i, t in enumerate(want_gemv):
                r = tm_rank[t]
                assert (cover[i, :r] == 1).all() and (cover[i, r:] <= 1).all() and (cover[i, (r + 7) // 8 * 8 :] == 0).all(), t
            cover = np.zeros((len(want_gemv), h_out), np.int8)
            for u in ge:
                same_entry(u)
                assert 0 <= u["lo"] < u["hi"] <= h_out and u["n_tok"] <= max_tok_e
                idx = [gemv_pos[int(t)] for t in toks_of(u)]
                assert len(set(idx)) == len(idx)
                cover[idx, u["lo"] : u["hi"]] += 1
            assert (cover == 1).all()

        gs = units[units["kind"] == B.LORA_UNIT_GEMV_SHRINK]
        ge = units[units["kind"] == B.LORA_UNIT_GEMV_EXPAND]
        covers_once(gs, ge, 4, 4, 4)
        assert sorted(gs["where"]) == list(range(len(gs)))
        for kinds, sizes in (((B.LORA_UNIT_BATCH_SHRINK, B.LORA_UNIT_BATCH_EXPAND), (4, 4, 4)),
                             ((B.LORA_UNIT_WIDE_SHRINK, B.LORA_UNIT_WIDE_EXPAND), (16, 8, 16))):
            bs, be = (units[units["kind"] == k] for k in kinds)
            entries = sorted(set(int(e) for e in bs["where"]))
            assert sorted(set(int(e) for e in be["where"])) == entries
            if not want_gemv or (not bf16 and sizes[0] == 16):
                assert not entries
                continue
            assert entries == [layer * len(projs) + p for layer in range(len(entries))] and 1 <= len(entries) <= 2
            for e in entries:
                covers_once(bs[bs["where"] == e], be[be["where"] == e], *sizes)

        # --- rows of the fused linear path: every token once, adapter tokens where the other lists have them
        lin = units[units["kind"] == B.LORA_UNIT_LINEAR_ROWS]
        if bf16:
            seen = np.zeros(T, np.int32)
            for u in lin:
                np.add.at(seen, toks_of(u), 1)
                assert 1 <= u["n_tok"] <= B.LORA_TILE_TOKENS
            assert (seen == 1).all()
            lt = lin[lin["where"] == 2]
            assert len(lt) == len(tiles)
            for u, v in zip(lt, tiles):
                assert list(toks_of(u)) == list(toks_of(v)) and (u["slot"], u["rank"], u["alpha"]) == (v["slot"], v["rank"], v["alpha"])
            g_rows = sorted(int(t) for u in lin[lin["where"] == 1] for t in toks_of(u))
            assert g_rows == want_gemv
            for u in lin[lin["where"] == 0]:
                assert (tm_slot[toks_of(u)] == -1).all()
        else:
            assert len(lin) == 0
        counts[p] = {"tiles": len(tiles), "gemv_shrink": len(gs), "gemv_expand": len(ge), "linear_rows": len(lin),
                     "tile_partial_sums": int((pieces["alpha"] >= 0).sum())}
    return counts
