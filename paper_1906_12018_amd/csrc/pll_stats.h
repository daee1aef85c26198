// What the phases of a batch count, per lane (plain C++: the functions run on
// the host as well).
#pragma once

namespace pll {

// One lane's counts of one round or batch end.  32 bits hold them: at up to
// 64 table quarters per label entry, a lane would have to read 2^26 entries
// in one round, i.e. its wave 2^32 (16 GiB of labels).  A kernel that runs
// many rounds takes the counts out after every round (take_counts) and keeps
// its sums in 64 bits.
struct PhaseStats {
    unsigned cand = 0, acc = 0, read = 0, table = 0, removed = 0, bp = 0;
    unsigned long long edges = 0;
    // cost of the positive / negative checks: |L(v)| at each check that
    // added / pruned a candidate (Section 4.3, Table 3)
    unsigned long long cost_pos = 0, cost_neg = 0;
    // CSR entries of the vertices whose next-round deliveries are pulled: the
    // edge accesses of Algorithm 4 (the gather itself reads more)
    unsigned long long pulled = 0;
};

// The counts the persistent kernels report, in this order.
enum { kCountCand, kCountAcc, kCountEdges, kCountRead, kCountTable, kCountRemoved, kCountPos, kCountNeg, kCounts };

// This lane's counts since the last call; st starts again at zero.
constexpr void take_counts(PhaseStats& st, unsigned long long (&v)[kCounts]) {
    v[kCountCand] = st.cand;
    v[kCountAcc] = st.acc;
    v[kCountEdges] = st.edges;
    v[kCountRead] = st.read;
    v[kCountTable] = st.table;
    v[kCountRemoved] = st.removed;
    v[kCountPos] = st.cost_pos;
    v[kCountNeg] = st.cost_neg;
    st = PhaseStats{};
}

}  // namespace pll
