"""Which forms the launch plans choose, and that the lists of the GPU tests reach the forms that they are there for."""
from plans import ask


def test_gemm_forms_on_either_side_of_the_line():
    """Sizes measured in both forms, us.  Counting even shares of the tokens alone, the direct form was taken where it is the slower
    one: 64 weight rows to a workgroup, or X the smaller part of what it takes in."""
    streamed = [(168, 3968, 2176), (36, 8064, 1536), (100, 4352, 1792), (46, 3968, 1920), (184, 3072, 1920), (255, 2688, 2688)]
    direct = [(1, 2560, 2048), (40, 2560, 2048), (192, 2048, 2048), (34, 1408, 1152), (66, 2176, 1408), (108, 1024, 2176), (36, 3328, 1536)]
    plans = ask(["gemm %d %d %d" % s for s in streamed + direct])
    assert [p["form"] == "direct" for p in plans] == [False] * len(streamed) + [True] * len(direct), plans


def test_gemm_forms_beside_two_token_parts():
    """Sizes measured in the direct form and in two token parts, us: 2560 x 2048 streams at every number of tokens (direct 14.2 at 150, 14.5 at
    160, 14.6 at 192, 16.8 at 240; in two parts 12.9, 13.1, 14.0, 15.9), few weight rows do not (200 x 2176 at 146 tokens 7.4 and 9.9)."""
    streamed = [(M, 2560, 2048) for M in (150, 160, 170, 176, 184, 188, 190, 191, 192, 193, 194, 196, 200, 208, 216, 224, 240)]
    streamed += [(192, 2304, 2048), (192, 2432, 2048), (192, 3072, 2048), (192, 2560, 1920), (192, 2560, 2176), (201, 1384, 3200), (252, 1336, 2432)]
    direct = [(134, 104, 2176), (146, 200, 2176), (182, 208, 2176), (143, 600, 2176), (173, 400, 2176), (148, 520, 2176), (135, 72, 2944)]
    plans = ask(["gemm %d %d %d" % s for s in streamed + direct])
    assert [p["form"] == "direct" for p in plans] == [False] * len(streamed) + [True] * len(direct), plans


def test_append_list_reaches_every_form():
    """Every tile of the direct form, K split in blocks of 64 and 128 rows, two token parts, and a product that streams W unsplit."""
    from test_gpu_gemm_append import SIZES
    plans = ask(["gemm %d %d %d" % (B * (k + 1), (Hq + 2 * Hkv) * D, K) for B, k, Hq, Hkv, D, K in SIZES])
    assert {(p["rn"], p["tt"]) for p in plans if p["form"] == "direct"} == {(1, 1), (1, 2), (2, 1), (2, 2), (2, 3), (4, 2), (4, 3)}
    assert {(p["form"], p["ksplit"] > 1) for p in plans if p["form"] != "direct"} == {("stream64", True), ("stream128", True), ("stream128", False)}


def test_short_sub_chunks_of_the_acceptance():
    from test_gpu_accept_parts import SHORT
    for (groups, parts, B, V), plan in zip(SHORT, ask(["accept %d %d" % c[2:] for c in SHORT])):
        assert (plan["groups"], plan["parts"]) == (groups, parts), (B, V, plan)
    # a row that one workgroup holds is not shared: there would be sums to exchange
    assert all(p["parts"] == 1 for p in ask(["accept %d %d" % (B, V) for B in (1, 4, 128) for V in (1, 257, 1000, 1024)]))


def attention(cfg):
    return "attention %d %d %d %d %d %d %d" % (cfg.B, cfg.k, cfg.Hq, cfg.Hkv, cfg.D, cfg.P, cfg.L)


def test_attention_lists_reach_the_one_tile_form_and_its_merges():
    from test_gpu_attention_items import ONE_TILE, ONE_TILE_MERGES, SEVERAL_TILES, TWO_ROW_TILES_D64
    plans = ask([attention(c) for c in ONE_TILE])
    for cfg, p in zip(ONE_TILE, plans):
        assert p["one"] == 1, (cfg, p)
    for nqt, merges in ONE_TILE_MERGES.items():
        assert {p["merge"] for p in plans if p["nqt"] == nqt} == merges, nqt
    assert any(p["fold"] for p in plans if p["merge"] == 4) and any(p["prefix_shares"] for p in plans if p["merge"] == 0)
    assert all(p["one"] == 0 for p in ask([attention(c) for c in SEVERAL_TILES]))
    assert all(p["nqt"] == 2 for p in ask([attention(c) for c in TWO_ROW_TILES_D64]))


def test_logits_lists_reach_every_size_of_piece():
    from test_gpu_logits_pieces import CASES
    from test_gpu_no_patience import LOGITS
    for case, p in zip(CASES, ask(["logits %d %d %d" % c[1:] for c in CASES])):
        assert p["loads"] == case[0], (case, p)
    assert {p["loads"] for p in ask(["logits %d %d %d" % c for c in LOGITS])} == {4, 5, 6, 8}


def test_lengths_lists_reach_the_flat_plan():
    """Small calls in the tests' build, long ones in the library itself: both merges, one row tile and two, with and without a prefix."""
    from test_gpu_attention_lengths import CASES, LONG, SHARED
    line = lambda c: attention(c).replace("attention", "lengths")
    plans = ask([line(c) for c in CASES], ("-DLOTTS_FLAT_STEPS=0",))
    assert all(p["flat"] for p in plans), list(zip(CASES, plans))
    assert {(c.D, p["nqt"], p["merge"]) for c, p in zip(CASES, plans)} == {(D, nqt, m) for D in (64, 128) for nqt in (1, 2) for m in (0, 1)}
    assert {p["fold"] for p in plans} == {0, 1} and 2 in {p["flat"] for p in plans}
    assert all(p["flat"] == 3 for p in ask([line(c) for c in SHARED], ("-DLOTTS_FLAT_STEPS=0",)))
    assert {p["merge"] for p in ask([attention(c) for c in SHARED])} == {0, 1, 3, 4}  # all that fixed shares of long calls have
    assert not any(p["flat"] for p in ask([line(c) for c in CASES]))
    long = ask([line(c) for c in LONG])
    assert all(p["flat"] == 1 for p in long) and {(p["nqt"], p["merge"]) for p in long} == {(1, 0), (1, 1), (2, 0), (2, 1)}
    # few bytes in fixed shares are no reason for the last arriver: a branch may have all items' partials
    assert long[4]["merge"] == 1 and ask([attention(LONG[4])])[0]["merge"] == 0
    # one branch more than a wavefront has lanes, rows of several row groups, a prefix in items of its own: not these
    other = [LONG[0].with_(B=65), LONG[0].with_(k=8), LONG[0].with_(P=LONG[0].L)]
    assert not any(p["flat"] for p in ask([line(c) for c in other]))


def test_a_buffer_for_more_branches_holds_fewer():
    """Where dealt tiles have more partials than the fixed shares of more branches, the fixed shares of the fewer fit: 64 branches of two KV heads
    ask for 4.9 MB, 128 for 3.3."""
    from synth_inputs import CONFIGS
    cfg = CONFIGS["C3"].with_(Hq=16, Hkv=2, k=2, P=1003, L=7168)
    few, many = ask([attention(cfg.with_(B=B)).replace("attention", "lengths") for B in (64, 128)])
    assert few["flat"] == 1 and not many["flat"]
    assert few["least"] <= many["bytes"] == many["least"] < few["bytes"]
    sizes = [cfg.with_(B=B, Hq=Hq, Hkv=Hkv, D=D, k=k, P=P, L=L) for B in (2, 7, 20, 40, 63) for Hq, Hkv, D in ((16, 2, 128), (40, 8, 128), (16, 16, 64))
             for k in (0, 3, 8) for P in (0, 500) for L in (2000, 16000)]
    plans = ask([attention(c).replace("attention", "lengths") for c in sizes])
    assert all(p["least"] <= p["bytes"] for p in plans) and sum(p["flat"] > 0 for p in plans) > 50
