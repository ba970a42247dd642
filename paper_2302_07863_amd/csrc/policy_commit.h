// The end of every pass with an LM head: fallback test, rollback test, commit, and what the host is told (policy.hip, pass_head.h).
#pragma once
#include "kernel_common.h"

namespace bild {

// The control words the policy needs.
struct Controls {
    int ylen, ds, nmax, len0, len1, lenw, seq;
    float afb, arb;
    unsigned turn;
    __device__ __forceinline__ explicit Controls(const FinishArgs& a) {
        const Ctl* c = a.ctl;
        ylen = c->y_len; ds = c->draft_start; nmax = c->n_max; len0 = c->len[0]; len1 = c->len[1]; lenw = c->len[a.which];
        afb = c->alpha_fb; arb = c->alpha_rb;
        seq = c->seq;
        turn = a.turn ? *a.turn : 0u;
    }
};

// By one wave, lane t with row t's statistics (argmax, max, sum of exp(z - max)).  The results go to the control block and,
// for the caller, to its mirror in pinned host memory (the words not written are the host's own).  The mirror is written
// past the caches and the pass counter once those stores have been acknowledged, so that a host that sees the new count also
// sees every other word.  (Volatile stores, one word after the other, each waited for its acknowledgement over the host
// link, and a system-wide fence writes the L2 back besides: 5 us for this kernel and 10 us for a wide one.)
// `failed`: the pass kernel's workgroups did not all run: nothing happened but the count of passes.  z_draft: logit of draft t; drawn: the
// sampling variant's token (-1: none); r_given: the first draft that the rejection rule refused (-1: the threshold decides).
// INSIDE: in the pass kernel itself (pass_head.h), whose counts go on; the flag of a failed pass stays for its workgroups that still wait (pass_gave_up).
template <bool INSIDE = false>
__device__ __forceinline__ void commit(const FinishArgs& a, const Controls& k, bool failed, int row_tok, float row_max, float row_sum, float z_draft, int drawn, int r_given) {
    const int lane = (int)threadIdx.x & 63, w = a.which, n = a.T - 1;
    Ctl* c = a.ctl;
    const int c_ylen = k.ylen, c_ds = k.ds, c_seq = k.seq;
    Ctl* v = a.host_mirror;
    const __amdgpu_buffer_rsrc_t mirror = make_rsrc(v, v ? sizeof(Ctl) : 0);  // (none: the stores are out of bounds and dropped)
    auto tell = [&](int word, int off) { __builtin_amdgcn_raw_buffer_store_b32((unsigned)word, mirror, off, 0, 17); };  // sc0 sc1
    float nll = 0.f, pmax = 0.f;
    if (a.mode != 3) {
        pmax = 1.f / row_sum;
        if (lane <= n) {
            c->res_rowtok[lane] = row_tok;
            tell(row_tok, (int)offsetof(Ctl, res_rowtok) + lane * 4);
        }
    }
    if (a.sync) {
        if (lane == 0 && a.turn) *a.turn = k.turn == 2u ? 0u : k.turn + 1u;
        if (!INSIDE && lane == 0) a.sync[0] = a.sync[kPassSyncWords - 1] = 0u;
        if (failed) {
            if (lane == 0) {
                c->seq = c_seq + 1;
                tell(kFlagFailed, (int)offsetof(Ctl, res_flag));
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) tell(c_seq + 1, (int)offsetof(Ctl, seq));
            return;
        }
    }
    int n_ylen = c_ylen, n_ds = c_ds, n_len0 = k.len0, n_lenw = k.lenw + a.rows_consumed;
    int res_tok = 0, res_flag = 0, res_r = 0, res_n = 0, y_at = -1;
    float res_pmax = 0.f;
    if (a.mode == 0 || a.mode == 2) {
        res_tok = drawn >= 0 ? drawn : __builtin_amdgcn_readlane(row_tok, n);
        res_pmax = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pmax), n));
        const bool low = a.mode == 0 && res_pmax < k.afb;
        const bool forced = a.mode == 0 && k.nmax > 0 && (c_ylen - c_ds) >= k.nmax;
        if (!low && !forced && c_ylen < a.y_cap) {
            y_at = c_ylen;
            n_ylen = c_ylen + 1;
            if (a.mode == 2) n_ds = c_ylen + 1;
        }
        res_flag = (low || forced ? 1 : 0) | ((forced && !low) ? 2 : 0);
    } else if (a.mode == 1) {  // review of n drafts: -ln p_L(draft) of each against the threshold
        nll = (row_max + logf(row_sum)) - z_draft;
        int r = r_given;       // (the rejection rule decided above)
        if (r < 0) {
            const unsigned long long over = __builtin_amdgcn_ballot_w64(lane < n && nll > k.arb);
            r = over ? (int)__builtin_ctzll(over) : n;
        }
        if (lane < n && (r_given < 0 || lane <= r)) {
            c->res_nll[lane] = nll;
            tell(__float_as_int(nll), (int)offsetof(Ctl, res_nll) + lane * 4);
        }
        res_tok = drawn >= 0 ? drawn : __builtin_amdgcn_readlane(row_tok, r);
        res_pmax = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pmax), r));
        y_at = c_ds + r;
        n_ylen = n_ds = c_ds + r + 1;
        n_lenw = c_ds + r;     // (w == 1)
        n_len0 = min(k.len0, c_ds + r);
        res_r = r;
        res_n = n;
    }
    const int l0 = w == 0 ? n_lenw : n_len0, l1 = w == 1 ? n_lenw : k.len1;
    const int sq = c_seq + 1;
    if (a.mode != 4) {
        if (lane == 0 && y_at >= 0) a.y[y_at] = res_tok;
        static_assert(offsetof(Ctl, res_tok) == 32 && offsetof(Ctl, res_pmax) == 48, "words 0 .. 3 and 8 .. 12");
        const int words[13] = {n_ylen, n_ds, l0, l1, 0, 0, 0, 0, res_tok, res_flag, res_r, res_n, __float_as_int(res_pmax)};
        int mine = 0;  // lane i has word i: one store
#pragma unroll
        for (int i = 0; i < 13; ++i) mine = lane == i ? words[i] : mine;
        if (lane < 13 && (lane < 4 || lane >= 8)) {
            tell(mine, lane * 4);
            ((int*)c)[lane] = mine;
        }
    }
    if (v) {
        static_assert(offsetof(Ctl, seq) == sizeof(Ctl) - 4, "seq must be the last word of the control block");
        if (lane == 0) c->seq = sq;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) tell(sq, (int)offsetof(Ctl, seq));
    }
}

}  // namespace bild
