"""Calls of fopd_lm_head_token_logprobs in which a workgroup's strip has several vocabulary tiles: rows, vocabulary, the form that
the launch takes and the rows of its whole token tiles.  Used on the card, and on the host to check that they are what they say."""

# one: all tokens in one tile of up to 384; narrow: all in one tile of up to 128; own: whole tiles of 256, and a last one of up to
# 128 with strips of its own; shared: the same with the strips of the others
STRIPS_OF_SEVERAL_TILES = [
    (257, 70001, "one", 0), (300, 70001, "one", 0), (384, 70001, "one", 0), (300, 32000, "one", 0), (372, 151936, "one", 0),
    (64, 151936, "narrow", 0), (128, 151936, "narrow", 0),
    (380, 151936, "own", 256), (600, 70001, "own", 512), (1100, 32000, "own", 1024),
    (1300, 32000, "shared", 1536),
]
