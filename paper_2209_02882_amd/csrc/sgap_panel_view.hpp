// What the kernels for long rows by column windows find in the caller's workspace.
#pragma once
#include <stdint.h>

namespace sgap {

constexpr int kRankMaxRows = 8192;     // lists up to this length are sorted by row length (every row looks at every other)

// How panel_lds_kernel's work is laid over the workgroups.
struct LdsPlan {
    uint32_t on;                // the kernel runs (those that gather through the L2 do not)
    uint32_t tiles, tile_cols;  // column tiles of B, columns of each (the last may have fewer)
    uint32_t groups, slots;     // groups of rows, rows of a team
    uint32_t per_die;           // shares of the columns that a die takes
    int32_t share_cols;         // columns of a share
    int32_t window;             // columns of a window
};

// The workspace: a header, the list of long rows, the same list sorted by length, the rows' lengths, and the
// window pointers.
struct PanelHeader {
    uint32_t count;     // long rows found (may exceed the list's capacity: then the path is off)
    uint32_t next[15];  // per die: the next item nobody has taken yet
    unsigned long long entries;  // stored entries of the rows found
    uint32_t nnz;                // of the matrix
    LdsPlan lds;
    uint32_t worst;            // the most of any row of those of:
    unsigned long long apart;  // entries of the rows found that windows in LDS would not serve, estimated
    uint32_t longest;          // entries of the longest of the rows found
    uint32_t pad[33];
};
struct PanelView {
    PanelHeader* head;
    int32_t* rows;   // [cap]
    int32_t* order;  // [cap] the long rows from the longest to the shortest: order[q] indexes rows[]
    int32_t* len;    // [cap] stored entries of rows[i]
    int32_t* ptr;    // [cap * (windows + 1)]: ptr[i * (windows + 1) + w] = first entry of long row i with column >= w * window_rows
    uint32_t cap;    // rows the list holds
};
static_assert(sizeof(PanelHeader) == 256, "the workspace's size is part of the interface");

// What the list of long rows is like.
struct LdsList {
    uint32_t count, longest, nnz, worst;  // nnz: of the matrix
    unsigned long long entries, apart;
};

// The choice between windows in LDS and gathers, worked out on the host (the device makes it by the same functions).
struct PanelForm {
    LdsPlan lds;
    float lds_clocks, gather_clocks;
};
PanelForm plan_panel_form(bool dots, int64_t K, int64_t N, const LdsList& list, int64_t window_bytes, bool window_asked,
                          int64_t cap, int xcds, int compute_units);

}  // namespace sgap
