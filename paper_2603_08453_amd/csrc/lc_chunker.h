// Structure-aware chunking (Section 4.3, Appendix B separator table) over any source of token texts:
// shared by the C entry point (one concatenated text) and the Python module (the str objects' own bytes).
#pragma once

#include <stdint.h>

#include "lychee.h"

struct LcTokenText {
    const char* p;
    int64_t len;
};

// 1 strongest .. 4 whitespace, 0 none.  One pass over the token's bytes: only a newline or a run of
// one of "-*`" makes a token a separator wherever it stands; everything else is decided by its end.
inline int lc_separator_level(const LcTokenText& t) {
    const char* const p = t.p;
    bool newline = false;
    for (int64_t i = 0; i < t.len; ++i) {
        const char c = p[i];
        if (c > '`') continue;                               // (most text bytes; bytes above 0x7f are negative)
        if (c == '\n') {
            if (i + 1 < t.len && p[i + 1] == '\n') return 1;
            newline = true;
        } else if (c == '-' || c == '*' || c == '`') {
            if (i + 2 < t.len && p[i + 1] == c && p[i + 2] == c) return 1;
        }
    }
    int64_t body = t.len;                                    // length without trailing blanks and tabs
    while (body > 0 && (p[body - 1] == ' ' || p[body - 1] == '\t')) --body;
    int at_end = 0;
    if (body > 0) {
        switch (p[body - 1]) {
            case '}': case ']': case '>': return 1;
            case '.': case '?': case '!': at_end = 2; break;
            case ',': case ';': case ':': at_end = 3; break;
            default:
                if ((unsigned char)p[body - 1] >= 0x80u && body >= 3) {     // full-width forms: three bytes each
                    const unsigned char a = (unsigned char)p[body - 3], b = (unsigned char)p[body - 2],
                                        c = (unsigned char)p[body - 1];
                    if (a == 0xE3u && b == 0x80u) at_end = c == 0x82u ? 2 : (c == 0x81u ? 3 : 0);
                    else if (a == 0xEFu && b == 0xBCu)
                        at_end = (c == 0x9Fu || c == 0x81u) ? 2 : ((c == 0x8Cu || c == 0x9Bu || c == 0x9Au) ? 3 : 0);
                }
        }
    }
    if (newline || at_end == 2) return 2;
    if (at_end == 3) return 3;
    return body < t.len ? 4 : 0;                             // ends in a blank (an all-blank token included)
}

// Greedy cut of n tokens: `level(i)` gives token i's separator level, `cut(end)` receives the end of every
// chunk in ascending order and returns false to stop.  Only the tokens in the search windows are looked at.
template <typename LevelF, typename CutF>
inline bool lc_chunk_cuts(int64_t n, int64_t min_len, int64_t max_len, LevelF level, CutF cut) {
    if (max_len > n) max_len = n;                            // (no chunk is longer than the text: the sums below stay in range)
    if (min_len > max_len) min_len = max_len;
    int64_t pos = 0;
    while (pos < n) {
        const int64_t hi = (pos + max_len < n ? pos + max_len : n) - 1;
        int64_t at = hi;
        int best = 5;
        for (int64_t e = pos + min_len - 1; e <= hi && best > 1; ++e) {
            const int lv = level(e);
            if (lv != 0 && lv < best) { best = lv; at = e; }
        }
        pos = at + 1;
        if (!cut(pos)) return false;
    }
    return true;
}
