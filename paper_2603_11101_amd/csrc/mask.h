// The masks as the kernels see them.  Plain integer code: it also compiles for the host, where it is checked against
// the definition of every mask.
#pragma once

#include "../../include/varlen_attn.h"

#ifndef VA_DEV
#define VA_DEV __device__ __forceinline__
#endif

namespace va {

// Every mask of the library has the form "local query row i sees keys j < vis(i)" with vis
// non-decreasing: causal i + 1; prefix-LM P for i < P, else L; prefix-LM with causal suffix P for
// i < P, else i + 1.  Branch-free so that it can sit in per-element code.
struct RowMask {
    int P;   // end of the first block (0 when causal)
    int P2;  // end of the second block (0 unless the mask has three blocks)
    int SF;  // L when the rows behind the blocks see the whole sample, else 0
    int L;
    VA_DEV RowMask(int item_P, int item_P2, int item_L, int mode)
        : P(item_P < 0 ? 0 : item_P),
          P2(item_P2 < 0 ? 0 : item_P2),
          SF(mode == VA_MASK_PREFIX_LM || mode == VA_MASK_THREE_BLOCK ? item_L : 0),
          L(item_L) {}
    // Every arm is computed before it is chosen, so that these stay selects and never become branches.
    VA_DEV int vis(int i) const {  // any i >= 0
        const int behind = max(i + 1, SF);
        const int second = i < P2 ? P2 : behind;
        return i < P ? P : second;
    }
};

// Every mask, the sliding window included, seen from both sides without branches: local query row i sees the keys
// lo(i) .. vis(i) - 1, and, since neither bound ever decreases, key j is seen by the rows first_row(j) .. end_row(j) - 1.
struct MaskBounds {
    RowMask upper;
    int width;  // of the sliding window; beyond any row for the other masks
    VA_DEV MaskBounds(int P, int P2, int L, int mode)
        : upper(mode == VA_MASK_SLIDING_WINDOW ? 0 : P, P2, L, mode), width(mode == VA_MASK_SLIDING_WINDOW ? P : 0x7fffffff) {}
    VA_DEV int vis(int i) const { return upper.vis(i); }
    VA_DEV int lo(int i) const { return max(0, i + 1 - width); }
    VA_DEV int first_row(int j) const {
        const int behind = upper.SF ? max(upper.P, upper.P2) : j;
        const int second = j < upper.P2 ? upper.P : behind;
        return j < upper.P ? 0 : second;
    }
    VA_DEV int end_row(int j) const { return width < upper.L ? min(upper.L, j + width) : upper.L; }
};

// The query rows as a wave of 32 keys jw .. jw + 31 sees them: those before some_from and from some_end on see none of
// its keys, those from all_from up to all_end - 1 all of them.  Keys past the sample count for neither, and a wave of
// nothing else is seen by no row (under the masks whose rows see whole samples it would otherwise compute every block:
// up to three of the four waves of a sample's last key tile).
struct KeyBlock {
    int some_from, some_end, all_from, all_end;
    VA_DEV KeyBlock(const MaskBounds& mask, int jw) {
        const int last_key = min(jw + 31, mask.upper.L - 1);
        some_from = mask.first_row(jw);
        some_end = jw < mask.upper.L ? mask.end_row(last_key) : 0;
        all_from = mask.first_row(last_key);
        all_end = mask.end_row(jw);
    }
};

}  // namespace va
