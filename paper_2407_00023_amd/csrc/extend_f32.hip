// Extend attention, fp32 arithmetic throughout (the tiny correctness configuration).
//
// The computation is the one the paper prices as "prefill of the missed tokens" with the
// cached prefix reused losslessly (Sec. 3.2, Sec. 5): extend row i of request r sees the
// P_r cached prefix tokens (rows of the pool named by slot_idx) and extend tokens 0..i.
//
// A workgroup computes the output rows of one extend token for up to kHeads query heads of one KV head.  D / 4 lanes
// share a key (16 bytes of its K row and of its V row each, so that rows are read whole and coalesced); the
// workgroup's 1,024 / D groups take keys in turn, each with an online softmax of its own, joined at the end.
// At the sizes this path serves (some hundred rows, some hundred keys) what bounds it is the chain of dependent memory
// round trips, not the arithmetic: a group's K and V rows are asked for together, kUnroll keys at a time, the slot ids
// of the next keys ahead of them, and the token's request is found by one comparison per lane instead of a search.
// (One wave per row, keys lane by lane, V row by row behind the scores: 28 us for 97 tokens x 4 heads over 96 keys.)
#include "common.h"

namespace pa {

// The request of extend token t: how many of ext_offsets[1 .. B) are <= t.
__device__ __forceinline__ int request_of(const int32_t* __restrict__ ext_offsets, int B, int64_t t) {
    constexpr int kDirect = 256;  // up to this many: all offsets in one round trip; beyond, a search
    if (B <= kDirect) {
        int r = 0;
#pragma unroll
        for (int c = 0; c < kDirect; c += 64) {
            const int k = c + static_cast<int>(threadIdx.x & 63);
            r += __popcll(__ballot(k >= 1 && k < B && ext_offsets[k] <= t));
        }
        return r;
    }
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (ext_offsets[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

template <int D, int kHeads>
__global__ __launch_bounds__(256) void extend_f32_kernel(
    const float* __restrict__ q_ext, const float* __restrict__ k_ext, const float* __restrict__ v_ext,
    const float* __restrict__ pool, const int32_t* __restrict__ slot_idx, const int32_t* __restrict__ slot_offsets,
    const int32_t* __restrict__ prefix_len, const int32_t* __restrict__ ext_len,
    const int32_t* __restrict__ ext_offsets, int B, int Hq, int Hkv, int page_size, int64_t num_slots,
    float scale, float* __restrict__ out) {
    constexpr int kLanes = D / 4;            // lanes of a group: one 16-byte piece of a row each
    constexpr int kGroups = 256 / kLanes;    // keys in work at once
    constexpr int kUnroll = 4;               // keys a group asks for together
    __shared__ float4 s_acc[4][kHeads][kLanes];
    __shared__ float s_m[4][kHeads], s_l[4][kHeads];
    const int tid = threadIdx.x, c = tid % kLanes, group = tid / kLanes;
    const int64_t t = blockIdx.x;
    const int G = Hq / Hkv, g = blockIdx.y;
    const int h0 = g * G + blockIdx.z * kHeads, n_heads = min(kHeads, (g + 1) * G - h0);

    // the token's request and what there is to know of it; up to 64 requests: all of it asked for together, a request per lane (us, one
    // after the other | together, 4 heads of 64: 4 requests, 95 tokens 6.52 | 6.27; 12, 433 tokens 21.0 | 20.7; 64, 994 tokens 17.6 | 16.8)
    int64_t e0;
    int P, E, slot_off;
    if (B <= 64) {
        const int lane = threadIdx.x & 63, k = min(lane, B - 1);
        const int o = ext_offsets[k], p = prefix_len[k], e = ext_len[k], so = slot_offsets[k];
        const int r = __popcll(__ballot(lane >= 1 && lane < B && o <= t));
        e0 = __builtin_amdgcn_readlane(o, r);
        P = __builtin_amdgcn_readlane(p, r);
        E = __builtin_amdgcn_readlane(e, r);
        slot_off = __builtin_amdgcn_readlane(so, r);
    } else {
        const int r = request_of(ext_offsets, B, t);
        e0 = ext_offsets[r];
        P = prefix_len[r];
        E = ext_len[r];
        slot_off = slot_offsets[r];
    }
    const int i = static_cast<int>(t - e0);
    const int32_t* __restrict__ slots = slot_idx + slot_off;
    if (i < 0 || i >= E) return;  // inconsistent offsets: produce nothing rather than read out of range
    const int nvis = P + i + 1;
    const unsigned last_slot = static_cast<unsigned>(min(num_slots, int64_t{INT32_MAX})) - 1u;

    float4 q[kHeads], acc[kHeads];
    float m[kHeads], l[kHeads];
#pragma unroll
    for (int x = 0; x < kHeads; ++x) {
        const float4 v = reinterpret_cast<const float4*>(q_ext + (t * Hq + h0 + min(x, n_heads - 1)) * D)[c];
        q[x] = make_float4(v.x * scale, v.y * scale, v.z * scale, v.w * scale);
        acc[x] = make_float4(0.f, 0.f, 0.f, 0.f);
        m[x] = -INFINITY;
        l[x] = 0.f;
    }
    // (keys past the end repeat the last visible one with probability 0: the lanes of a group stay together)
    auto slot_of = [&](int j) { return j < P ? slots[j] : 0; };
    int32_t sl[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) sl[u] = slot_of(min(u * kGroups + group, nvis - 1));
    for (int j0 = 0; j0 < nvis; j0 += kGroups * kUnroll) {
        float4 k[kUnroll], v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int j = min(j0 + u * kGroups + group, nvis - 1);
            const float *kp, *vp;
            if (j < P) {
                const unsigned s = min(static_cast<unsigned>(max(sl[u], 0)), last_slot);  // never outside the pool
                const unsigned page = s / static_cast<unsigned>(page_size), o = s - page * static_cast<unsigned>(page_size);
                const int64_t row = (static_cast<int64_t>(page) * 2 * Hkv + g) * page_size + o;
                kp = pool + row * D;
                vp = kp + static_cast<int64_t>(Hkv) * page_size * D;
            } else {
                const int64_t row = (e0 + (j - P)) * Hkv + g;
                kp = k_ext + row * D;
                vp = v_ext + row * D;
            }
            k[u] = reinterpret_cast<const float4*>(kp)[c];
            v[u] = reinterpret_cast<const float4*>(vp)[c];
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) sl[u] = slot_of(min(j0 + (kUnroll + u) * kGroups + group, nvis - 1));
#pragma unroll
        for (int x = 0; x < kHeads; ++x) {
            float s[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                float d = q[x].x * k[u].x + q[x].y * k[u].y + q[x].z * k[u].z + q[x].w * k[u].w;
#pragma unroll
                for (int off = 1; off < kLanes; off <<= 1) d += __shfl_xor(d, off);
                s[u] = j0 + u * kGroups + group < nvis ? d : -INFINITY;
            }
            // (a key past the end has probability 0, which must not meet an infinity of the row it repeats; here and not at the
            // loads, so that the scores do not wait for the V rows)
            if (x == 0 && j0 + kGroups * kUnroll > nvis)
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    if (j0 + u * kGroups + group >= nvis) v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            float mx = m[x];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) mx = fmaxf(mx, s[u]);
            const float ref = mx == -INFINITY ? 0.f : mx;  // (a group that has seen no key yet)
            const float alpha = expf(m[x] - ref);
            m[x] = mx;
            l[x] *= alpha;
            acc[x].x *= alpha; acc[x].y *= alpha; acc[x].z *= alpha; acc[x].w *= alpha;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const float p = expf(s[u] - ref);
                l[x] += p;
                acc[x].x += p * v[u].x; acc[x].y += p * v[u].y; acc[x].z += p * v[u].z; acc[x].w += p * v[u].w;
            }
        }
    }
    // join the groups: those of a wave by exchange, then the four waves through LDS
    const int wave = tid >> 6, lane = tid & 63;
#pragma unroll
    for (int x = 0; x < kHeads; ++x) {
#pragma unroll
        for (int off = kLanes; off < 64; off <<= 1) {
            const float mo = __shfl_xor(m[x], off), mn = fmaxf(m[x], mo), ref = mn == -INFINITY ? 0.f : mn;
            const float a = expf(m[x] - ref), b = expf(mo - ref);
            l[x] = l[x] * a + __shfl_xor(l[x], off) * b;
            acc[x].x = acc[x].x * a + __shfl_xor(acc[x].x, off) * b;
            acc[x].y = acc[x].y * a + __shfl_xor(acc[x].y, off) * b;
            acc[x].z = acc[x].z * a + __shfl_xor(acc[x].z, off) * b;
            acc[x].w = acc[x].w * a + __shfl_xor(acc[x].w, off) * b;
            m[x] = mn;
        }
        if (lane < kLanes) s_acc[wave][x][c] = acc[x];
        if (lane == 0) {
            s_m[wave][x] = m[x];
            s_l[wave][x] = l[x];
        }
    }
    __syncthreads();
    for (int y = tid; y < n_heads * D; y += 256) {
        const int x = y / D, d = y % D;
        float mx = s_m[0][x];
#pragma unroll
        for (int w = 1; w < 4; ++w) mx = fmaxf(mx, s_m[w][x]);
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float a = expf(s_m[w][x] - mx);  // (some group has seen key 0, so the maximum is finite)
            num += a * reinterpret_cast<const float*>(&s_acc[w][x][0])[d];
            den += a * s_l[w][x];
        }
        out[(t * Hq + h0 + x) * D + d] = num / den;
    }
}

}  // namespace pa

// Called by pa_extend_attention after argument validation.
int pa_extend_attention_f32(const void* q_ext, const void* k_ext, const void* v_ext, const void* kv_pool,
                            const int32_t* slot_idx, const int32_t* slot_offsets, const int32_t* prefix_len,
                            const int32_t* ext_len, const int32_t* ext_offsets, int B, int64_t T, int Hq, int Hkv, int D,
                            int page_size, int64_t num_slots, float scale, void* out, hipStream_t stream) {
    // query heads a workgroup takes at once: all of a KV head's up to four (they share its K and V rows)
    const int G = Hq / Hkv, per_wg = G >= 3 ? 4 : G;
    PA_REQUIRE(Hkv <= 65535 && (G + per_wg - 1) / per_wg <= 65535, "pa_extend_attention: too many heads (%d, %d)", Hq, Hkv);
    const dim3 grid(static_cast<unsigned>(T), static_cast<unsigned>(Hkv), static_cast<unsigned>((G + per_wg - 1) / per_wg)), block(256);
#define PA_LAUNCH_F32(DD, HH)                                                                                    \
    hipLaunchKernelGGL((pa::extend_f32_kernel<DD, HH>), grid, block, 0, stream, static_cast<const float*>(q_ext), \
                       static_cast<const float*>(k_ext), static_cast<const float*>(v_ext),                       \
                       static_cast<const float*>(kv_pool), slot_idx, slot_offsets, prefix_len, ext_len,          \
                       ext_offsets, B, Hq, Hkv, page_size, num_slots, scale, static_cast<float*>(out))
    {
        pa::ProfScope prof(pa::kProfExtendF32, stream);
        if (D == 64 && per_wg == 1) PA_LAUNCH_F32(64, 1);
        else if (D == 64 && per_wg == 2) PA_LAUNCH_F32(64, 2);
        else if (D == 64) PA_LAUNCH_F32(64, 4);
        else if (per_wg == 1) PA_LAUNCH_F32(128, 1);
        else if (per_wg == 2) PA_LAUNCH_F32(128, 2);
        else PA_LAUNCH_F32(128, 4);
    }
#undef PA_LAUNCH_F32
    PA_HIP(hipGetLastError());
    return PA_OK;
}
