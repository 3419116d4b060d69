"""Launch configuration of each measured workload: lanes per station of every
class, waves per block and the observation stage -- the fastest found on
MI355X by timing every legal choice on that workload.  bench.py times each
workload in exactly this configuration and the full-size parity tests run it,
so what is measured is what is checked."""
from __future__ import annotations

# Waves up to which several packings run as one launch, which has no observation
# stage and is the faster there (the uneven mixture, 288 steps, every record: 2,000
# stations 0.49 ms against 0.80, 20,000 1.16 against 1.20, 28,000 1.58 against 1.52).
SHARED_LAUNCH_WAVES = 10240
# workload -> (lanes per station, or None for every class at min(slots, 64);
#              waves per block; observation stage past SHARED_LAUNCH_WAVES)
LAUNCH = {
    "uneven-batching": (None, 4, True),
    "v2g": (8, 1, False),
    "users": (8, 1, False),
    "exo": (8, 1, False),
    "tiny": (16, 1, False),
    "scale": (16, 1, False),
}
# The policy rollout of a SIMPLE class of 8, 16 or 32 slots is the fused kernel,
# whose launch is fixed (4 waves per block; 8 lanes per station, or 16 for 16-slot
# stations while every block has a CU of its own), as is that of a general class
# packed with one slot per lane; this packing of the policy workload's SIMPLE class
# serves the two-kernel path, which the rollout that allocates nothing takes
# (8 lanes x 4 slots, 4 waves per block).
POLICY_LAUNCH = (8, 4)


def configure(env, workload: str, n_classes: int) -> None:
    """Set the packing of every class and the stage of ``env`` for ``workload``
    (a key of LAUNCH, or a description that opens with one and a colon)."""
    lanes, wpb, stage = LAUNCH[workload.split(":")[0]]
    waves = 0
    for c in range(n_classes):
        ci = env.class_info(c)
        L = lanes if lanes is not None else min(ci.slots, 64)
        env.set_packing(c, L, wpb)
        groups = -(-ci.n_envs // (64 // L))
        waves += -(-groups // wpb) * wpb
    env.set_obs_stage(stage and waves > SHARED_LAUNCH_WAVES)
