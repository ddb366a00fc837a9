// How the CG kernels read the iteration at which a run stops.
//
// The stop of iteration k is recorded (stop_at = k) inside the launch that
// opens iteration k, by one block, while the other blocks of that launch are
// still reading the state.  A wave may therefore see stop_at = k or the value
// from before the launch, and the waves of one block may differ.  So nothing in
// that launch may depend on which of the two it saw: only stop_at < k, which no
// block of it can write, lets a wave leave ahead of a barrier, and stop_at = k
// decides after the block's sum, where the same sum stops every wave.
// Plain C++, so that the rule can be run over all interleavings on the host.
#pragma once

namespace fgi {

// Opening of iteration iter by the classic form's direction update: whether the
// wave goes on to update p, and the beta it takes.  sum() is the block's sum of
// the |r|^2 partials, with barriers (every wave of the block must call it, or
// none); record(rr, beta, stop) writes the state and is called by the one
// thread with `first` set.
template <typename State, typename Sum, typename Record>
constexpr bool cg_open(const State& S, int iter, bool first, Sum sum, Record record, double& beta) {
    if (S.stop_at < iter) return false;
    beta = S.beta;
    if (iter != S.base0) {
        const double rr = sum();
        const bool stop = rr <= S.rr_stop;
        beta = rr / ((iter & 1) ? S.rr[0] : S.rr[1]);   // |r|^2 of iteration iter - 1
        if (first && S.stop_at > iter) record(rr, beta, stop);
        if (stop) return false;
    }
    return S.stop_at > iter;
}

// Whether a block of any other CG kernel has nothing to do.  opens: a site block
// of the hop that opens a Chronopoulos-Gear iteration, whose reduction block
// records the stop beside it (its output is scratch, so it just goes on).
constexpr bool cg_leaves(int stop_at, int iter, bool opens) { return opens ? stop_at < iter : stop_at <= iter; }

// Where an inner run that began at iteration base0 is cut off: after the whole
// batches that reach maxiter (any maxiter up to the largest int; the sum past it
// stays there).
constexpr int cg_cut(int base0, int maxiter, int batch) {
    const long long left = (long long)maxiter - base0;
    const long long cut = base0 + (left + batch - 1) / batch * batch;
    return cut < 0x7fffffff ? (int)cut : 0x7fffffff;
}

}  // namespace fgi
