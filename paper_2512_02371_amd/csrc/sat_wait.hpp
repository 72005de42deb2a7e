// The grid-wide wait of hb_sat2d's one-launch kernel: its words in the workspace and the steps that one lane of a workgroup takes.
// The accesses to memory are a parameter, so that the tests run these very steps with threads as workgroups.
//
// Arrival is a two-level count (up to 16 leaf counters, one root, each on its own
// 128-byte line: arrivals at one address are served one after the other by the memory side); the
// last arrival raises eight copies of a `go` word and workgroup w polls copy w % 8.  Table data and
// the words of the wait are written and read with agent-scope accesses (they bypass the per-XCD L2,
// so no cache write-back or invalidation is needed; a write-back per workgroup costs ~20 ns each,
// one after the other).  The wait is BOUNDED: after `wait_limit` polls a workgroup stops waiting.
// It has already arrived, so the count still completes when the last workgroup gets to run; a
// workgroup that stopped waiting marks its region in `todo`, raises `late` and leaves, unless `go`
// came up meanwhile.  Every workgroup that passes the wait reads `late` (raised before `go` by
// construction, see below) and, if it is set, claims marked regions one by one, reloads their
// pixels and finishes them.  So every wave exits whatever the residency, and every region is
// finished by someone:
//   late workgroup: store todo[r], late; wait for the stores; load go.  go == 0 -> leave.
//   finisher:       observes go == 1; then loads late and todo.
//   go is raised once, after the late workgroup's load returned 0, hence after its stores were
//   performed at the memory side: the finisher's loads see them.  (That holds for the workgroup that raised `go`, whose own
//   poll of it waits for all its stores; another one may find one copy up before the next is.)
// With two groups, `go` of the first, once performed, counts as one more arrival of the second, so `go` of the second
// means that every region is published.  A workgroup finishes only regions that it knows to be: those of the first group,
// and all of them if it is of the second or raised the second's `go` itself.  (The workgroup that raises a group's `go`
// always passes its own wait, so some workgroup finishes what that group's late ones left.)
//
// The words of the wait hold anything when the kernel starts.  The launch's number `call` (unlike any other launch's) tells
// whether they are this launch's: workgroup 0 exchanges it for `claim`, clears the words if it was the first, and then writes it
// to `ready`, which every workgroup has to find there before it arrives; one that has looked for long does the clearing
// itself, through the same exchange.  This look is not subject to `wait_limit` (who leaves before it arrives is missed by all the
// others), but it waits for no workgroup that does not run: whoever won `claim` is running, and does nothing that waits before it sets
// `ready`.  Only words that something else writes meanwhile, a second launch with the same workspace, can keep it
// from coming; for that case it ends after kReadyPolls, about two seconds, and so does the kernel, with its table incomplete.
// The last arrival of all wipes `claim` and `ready`, which nobody reads from then on: a launch that is replayed from a
// graph with the same number finds its words not ready again.
#pragma once

namespace hb {

struct SatSync {
    static constexpr int kLine = 32;                      // words per 128 bytes
    static constexpr int kLeaves = 16, kGo = 8, kMaxRegions = 1024;     // leaves and copies of `go`: halved between two groups
    static constexpr int kRoot = 16;                      // words from the first group's root to the second's
    static constexpr int kReady = 8, kClaim = 8;          // words at which the lines of `go` and `late` have `ready` and `claim`
    unsigned leaf[kLeaves * kLine];
    unsigned root[kLine];
    unsigned go[kGo * kLine];                             // each copy with one of `ready` (64 bits)
    unsigned late[kLine];                                 // with `claim` (64 bits)
    unsigned todo[kMaxRegions];                           // 0 idle, 1 waiting for a finisher, 2 claimed
#ifdef HB_SAT_TIMING
    unsigned long long stamp[kMaxRegions][8];             // measurement builds only: phase time stamps per workgroup
#endif
};

constexpr int kSatClaimPolls = 64;                        // of `ready`, after which a workgroup offers to clear
constexpr int kSatReadyPolls = 1 << 21;                   // ... after which it gives up

// Mem: load and store of a word or a 64-bit number, add (the new value), exchange (the old value), claim (1 -> 2, whether it
// did), performed (all earlier stores are), pause (between two polls).
template <class Mem>
struct SatWait {
    using Call = unsigned long long;
    static __device__ __forceinline__ Call* ready(SatSync* s, int copy) {
        return reinterpret_cast<Call*>(&s->go[SatSync::kLine * copy + SatSync::kReady]);
    }
    static __device__ __forceinline__ Call* claim(SatSync* s) { return reinterpret_cast<Call*>(&s->late[SatSync::kClaim]); }
    // By the last arrival of all, when nobody reads these any more: leaves no trace of this launch's number.
    static __device__ __forceinline__ void forget_call(SatSync* s) {
        for (int i = 0; i < SatSync::kGo; ++i) Mem::store(ready(s, i), Call(0));
        Mem::store(claim(s), Call(0));
    }
    // Taking on the clearing of the wait's words: whether no other workgroup of this launch has.
    static __device__ __forceinline__ bool take(SatSync* s, Call call) { return Mem::exchange(claim(s), call) != call; }
    // Lanes 0 .. n - 1 of one wave: the clearing, and, once that is performed, `ready`.
    static __device__ __forceinline__ void clear(SatSync* s, int nwg, int lane, int n) {
        for (int i = lane; i < SatSync::kLeaves; i += n) Mem::store(&s->leaf[SatSync::kLine * i], 0u);
        for (int i = lane; i < SatSync::kGo; i += n) Mem::store(&s->go[SatSync::kLine * i], 0u);
        for (int i = lane; i < 2; i += n) Mem::store(&s->root[SatSync::kRoot * i], 0u);
        if (lane == 0) Mem::store(&s->late[0], 0u);
        for (int i = lane; i < nwg; i += n) Mem::store(&s->todo[i], 0u);
    }
    static __device__ __forceinline__ void set_ready(SatSync* s, Call call, int lane, int n) {
        Mem::performed();
        for (int i = lane; i < SatSync::kGo; i += n) Mem::store(ready(s, i), call);
    }

    // One lane of workgroup wg, whose region is published: arrives and waits.  0: leave (someone else finishes the region);
    // passed, and published are: 1 the first group's regions, 2 all.  first: workgroups of the first group, nwg if there is no other.
    static __device__ __forceinline__ int arrive(SatSync* S, int wg, int nwg, int first, Call call, int wait_limit, int claim_polls) {
        Call* const mine = ready(S, wg & (SatSync::kGo - 1));
        for (int polls = 0; Mem::load(mine) != call; ++polls) {
            if (polls == claim_polls && take(S, call)) {
                clear(S, nwg, 0, 1);
                set_ready(S, call, 0, 1);
            }
            if (polls == kSatReadyPolls) return 0;
            Mem::pause();
        }
        const int ngroups = first < nwg ? 2 : 1, group = wg < first ? 0 : 1;
        const int kl = SatSync::kLeaves / ngroups, kg = SatSync::kGo / ngroups;
        const int id = group ? wg - first : wg, n1 = nwg - first, n = group ? n1 : first;
        const int nleaf = n < kl ? n : kl, lf = id % nleaf;
        const int leaf_target = (n - lf + nleaf - 1) / nleaf;
        bool all = ngroups == 1 || group == 1;            // passing the wait, it knows that every region is published
        auto raise = [&](int g) {
            for (int i = 0; i < kg; ++i) Mem::store(&S->go[SatSync::kLine * (g * kg + i)], 1u);
            if (g == ngroups - 1) forget_call(S);
        };
        if ((int)Mem::add(&S->leaf[SatSync::kLine * (group * kl + lf)]) == leaf_target &&
            (int)Mem::add(&S->root[SatSync::kRoot * group]) == nleaf + group) {
            raise(group);
            if (ngroups == 2 && group == 0) {             // the first group is one more arrival of the second
                Mem::performed();
                if ((int)Mem::add(&S->root[SatSync::kRoot]) == (n1 < kl ? n1 : kl) + 1) {
                    raise(1);
                    all = true;
                }
            }
        }
        const unsigned* const mygo = &S->go[SatSync::kLine * (group * kg + id % kg)];
        const int passed = all ? 2 : 1;
        for (int polls = 0; Mem::load(mygo) == 0u;) {
            if (++polls > wait_limit) {                   // stop waiting: hand the region to a finisher
                Mem::store(&S->todo[wg], 1u);
                Mem::store(&S->late[0], 1u);
                Mem::performed();
                if (Mem::load(mygo) == 0u) return 0;
                Mem::claim(&S->todo[wg]);                 // the count completed meanwhile: finish it here after all
                return passed;                            // (a finisher may have claimed it too: both write the same values)
            }
            Mem::pause();
        }
        return passed;
    }
};

}  // namespace hb
