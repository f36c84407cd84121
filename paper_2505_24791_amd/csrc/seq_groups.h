// Groups of the persistent sequential kernel: which workgroups carry which samples.  Plain C++ beside the kernel, so that the
// arithmetic can be checked without a device.
#pragma once

#ifdef __HIPCC__
#define SJD_HOST_DEVICE __host__ __device__
#else
#define SJD_HOST_DEVICE
#endif

namespace sjd {

struct SeqGroup {
    int index, groups;     // this group, groups in all
    int members, before;   // workgroups of the group, those of them on lower XCDs than the caller's
    int per;               // samples per group (the last groups may have fewer, or none)
};

// The group of the workgroups on XCD `xcc` when count[] workgroups run on each of the eight XCDs: `xpg` neighbouring XCDs that have
// any form a group.  The host chooses xpg for a device of eight XCDs; with fewer (a partition of the device) it is halved until a group's
// share of the B samples is at most max_rows, which is as far as one XCD per group goes.
SJD_HOST_DEVICE inline SeqGroup seq_group_of(const int (&count)[8], int xcc, int xpg, int B, int max_rows) {
    SeqGroup g{};
    int rank = 0, present = 0;
    for (int x = 0; x < 8; ++x) {
        if (x == xcc) rank = present;
        present += count[x] > 0 ? 1 : 0;
    }
    for (;; xpg /= 2) {
        g.groups = (present + xpg - 1) / xpg;
        g.per = (B + g.groups - 1) / g.groups;
        if (g.per <= max_rows || xpg == 1) break;
    }
    g.index = rank / xpg;
    int seen = 0;
    for (int x = 0; x < 8; ++x) {
        if (count[x] <= 0) continue;
        if (seen / xpg == g.index) {
            g.members += count[x];
            if (x < xcc) g.before += count[x];
        }
        ++seen;
    }
    return g;
}

}  // namespace sjd
