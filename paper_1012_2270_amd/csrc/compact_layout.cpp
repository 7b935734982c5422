// Host side of the compact column storage (compact.h): the pattern search and
// the x windows of a host layout.  Plain C++17; no device code.
#include <algorithm>
#include <cstring>
#include <unordered_map>

#include "compact.h"

namespace rg {

namespace {

// (constants: the golden ratio, and the first multiplier of the published
// MurmurHash3 64-bit finalizer)
uint64_t mix(uint64_t h, uint64_t v) {
    h ^= v + 0x9e3779b97f4a7c15ull + (h << 6) + (h >> 2);
    h *= 0xff51afd7ed558ccdull;
    return h ^ (h >> 32);
}

// Row patterns of the layout; false when the rows need more than kPatMax
// lists or a table that does not pay.
bool find_patterns(const HostLayout &L, HostCompact &C) {
    std::vector<std::vector<int32_t>> lists;
    std::unordered_map<uint64_t, int32_t> seen;
    std::vector<int32_t> cur, step, differs;
    int32_t longest = 0, last = -1;
    C.pat_id.resize((size_t)L.ns);
    for (int64_t g = 0; g < L.ng; g++) {
        const int64_t r0 = L.ragged ? L.grp_row0[g] : g * L.G;
        const int64_t r1 = L.ragged ? L.grp_row0[g + 1] : std::min<int64_t>(L.ns, r0 + L.G);
        const int64_t sg = r1 - r0;
        const int64_t width = sg ? (L.group_end(g) - L.gp[g]) / sg : 0;
        if (width > kPatLen) return false;
        // Neighbouring rows mostly share a list: a row of the length before it
        // whose columns are all as far from that row's as the rows are apart
        // (padding repeats the last column), told step by step, rows side by
        // side as they lie (1.8M nonzeros: row by row 3.4 ms).
        step.assign((size_t)sg, 0);
        differs.assign((size_t)sg, 1);
        for (int64_t i = 1; i < sg; i++) {
            step[i] = L.short_row[r0 + i] - L.short_row[r0 + i - 1];
            differs[i] = L.short_len[r0 + i] != L.short_len[r0 + i - 1];
        }
        for (int64_t j = 0; j < width; j++) {
            const int32_t *c = &L.slot_col[L.gp[g] + j * sg], *st = step.data();
            int32_t *df = differs.data();
            for (int64_t i = 1; i < sg; i++) df[i] |= (uint32_t)c[i] - (uint32_t)c[i - 1] != (uint32_t)st[i];
        }
        for (int64_t i = r0; i < r1; i++) {
            if (!differs[i - r0]) {
                C.pat_id[i] = (uint8_t)last;
                continue;
            }
            const int32_t len = L.short_len[i];
            const int64_t row = L.short_row[i], s0 = L.gp[g] + (i - r0);
            cur.resize(len);
            uint64_t h = mix(0, (uint64_t)len);
            for (int32_t j = 0; j < len; j++) {
                const int64_t d = (int64_t)L.slot_col[s0 + j * sg] - row;
                cur[j] = (int32_t)d;
                h = mix(h, (uint64_t)d);
            }
            auto it = seen.find(h);
            if (it == seen.end()) {
                longest = std::max(longest, len);
                if ((int)lists.size() == kPatMax ||
                    !pat_pays((int64_t)lists.size() + 1, pat_stride(longest), L.slots))
                    return false;
                it = seen.emplace(h, (int32_t)lists.size()).first;
                lists.push_back(cur);
            } else if (lists[it->second] != cur) {
                return false;  // two lists of one hash: not worth a second search
            }
            last = it->second;
            C.pat_id[i] = (uint8_t)last;
        }
    }
    C.n_pat = (int32_t)lists.size();
    C.stride = pat_stride(longest);
    C.pat_tab.assign((size_t)C.n_pat * C.stride, 0);
    for (int32_t p = 0; p < C.n_pat; p++) {
        int32_t *t = &C.pat_tab[(size_t)p * C.stride];
        t[0] = (int32_t)lists[p].size();
        std::copy(lists[p].begin(), lists[p].end(), t + 1);
    }
    C.segs = pattern_segments(C.pat_tab.data(), C.n_pat, C.stride);
    return true;
}

}  // namespace

// Runs of offsets with gaps of at most 64; none where they are more than
// kPatSegs, or their entries do not fit one load of the ends and the buffer.
PatSegs pattern_segments(const int32_t *tab, int32_t n_pat, int32_t stride) {
    std::vector<int32_t> off;
    for (int32_t p = 0; p < n_pat; p++) {
        const int32_t *t = tab + (size_t)p * stride;
        off.insert(off.end(), t + 1, t + 1 + t[0]);
    }
    std::sort(off.begin(), off.end());
    PatSegs S;
    for (size_t i = 0; i < off.size(); i++) {
        if (i == 0 || (int64_t)off[i] - off[i - 1] > 64) {
            if (S.n == kPatSegs) return PatSegs();
            S.lo[S.n++] = off[i];
        }
        S.span[S.n - 1] = off[i] - S.lo[S.n - 1];
    }
    for (int32_t s = 0; s < S.n; s++) {
        S.base[s] = S.total;
        S.total += kBlockThreads + S.span[s];
        S.extra += S.span[s];
    }
    for (int32_t s = S.n; s > 0 && s < kPatSegs; s++) {
        S.lo[s] = S.lo[s - 1];
        S.base[s] = S.base[s - 1];
    }
    if (S.n == 0 || S.extra > kBlockThreads || S.total > kWinCols) return PatSegs();
    return S;
}

namespace {

// x windows of the layout's units; false when some unit's columns span more
// than kWinCols or the windows do not pay.
bool find_windows(const HostLayout &L, HostCompact &C) {
    const int64_t per = (int64_t)kBlockWaves * C.rows;
    const int64_t units = (L.ng + per - 1) / per;
    C.win.assign((size_t)(2 * units), 0);
    int64_t total = 0;
    for (int64_t u = 0; u < units; u++) {
        int64_t lo = INT32_MAX, hi = -1;
        for (int64_t g = u * per; g < std::min(L.ng, (u + 1) * per); g++) {
            const int64_t r0 = L.ragged ? L.grp_row0[g] : g * L.G;
            const int64_t r1 = L.ragged ? L.grp_row0[g + 1] : std::min<int64_t>(L.ns, r0 + L.G);
            const int64_t width = r1 > r0 ? (L.group_end(g) - L.gp[g]) / (r1 - r0) : 0;
            if (width == 0) continue;
            // a row's first column lies in the first step and its last one in
            // the last (padding repeats it; 0 for an empty row)
            const int32_t *first = &L.slot_col[L.gp[g]], *final = first + (width - 1) * (r1 - r0);
            for (int64_t i = 0; i < r1 - r0; i++) {
                if (L.short_len[r0 + i]) lo = std::min<int64_t>(lo, first[i]);
                hi = std::max<int64_t>(hi, final[i]);
            }
        }
        if (hi < 0) continue;  // a unit of empty rows
        if (hi - lo >= kWinCols) return false;
        C.win[2 * u] = (int32_t)lo;
        C.win[2 * u + 1] = (int32_t)(hi - lo + 1);
        total += hi - lo + 1;
    }
    if (!win_pays(total, L.slots, L.nnz)) return false;
    C.col16.assign((size_t)L.slots, 0);
    for (int64_t g = 0; g < L.ng; g++) {
        const int32_t base = C.win[2 * (g / per)];
        const int64_t end = L.group_end(g);
        const int32_t *c = L.slot_col.data();
        uint16_t *o = C.col16.data();
        for (int64_t s = L.gp[g]; s < end; s++) o[s] = (uint16_t)std::max(c[s] - base, 0);
    }
    return true;
}

}  // namespace

void build_compact(const HostLayout &L, HostCompact &C) {
    C = HostCompact();
    if (L.T != 1 || L.G % 64 != 0 || L.nl > 0 || L.ns == 0) return;
    if (find_patterns(L, C)) {
        C.mode = kCompactPattern;
        C.width = C.stride - 1;
        C.rows = compact_rows(C.width, L.esz);
        return;
    }
    C = HostCompact();
    if (L.G != 64 || L.slots < kWinMinSlots) return;
    C.rows = compact_rows(L.slots / L.ns, L.esz);
    if (find_windows(L, C)) {
        C.mode = kCompactWindow;
        return;
    }
    C = HostCompact();
}

}  // namespace rg
